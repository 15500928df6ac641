// Khatri-Rao reductions, flat reductions and layout kernels.
#include "kernels.hpp"

namespace tk {

namespace {

struct Dims4 {
  int v[kMaxD];
};

constexpr int KRP_NT = 256;
constexpr int KRP_ZMAX = 128;

// One workgroup per (column l, task).  M_j[:, l] is staged in LDS; threads
// split the contraction over the non-free multi-index and combine partial
// sums in a fixed order (bitwise reproducible).
template <typename T>
__global__ __launch_bounds__(KRP_NT) void krp_kernel(const KrpTask<T>* __restrict__ tasks, int m, Dims4 z,
                                                     int P, int S) {
  __shared__ T mv[kMaxD][KRP_ZMAX];
  __shared__ T part[KRP_NT];
  const int l = blockIdx.x;
  const KrpTask<T> tk_ = tasks[blockIdx.y];
  const int f = tk_.f, ldo = tk_.ldo;
  const int tid = threadIdx.x;
#pragma unroll
  for (int j = 0; j < kMaxD; ++j) {
    if (j >= m || j == f) continue;
    for (int i = tid; i < z.v[j]; i += KRP_NT) mv[j][i] = tk_.Mj[j][i + (size_t)l * tk_.ldm[j]];
  }
  __syncthreads();
  const T* Zl = tk_.Z + (size_t)l * P;
  double coef = tk_.scale * (tk_.coef ? *tk_.coef : 1.0);
  if (f >= 0) {
    const int zf = z.v[f];
    const int nparts = KRP_NT / zf;
    const int a = tid % zf, pp = tid / zf;
    const int O = P / zf;
    T acc = T(0);
    if (pp < nparts) {
      // strides of the row-major multi-index (loops over the fixed kMaxD
      // modes, unrolled, so that the index arrays stay in registers)
      int stride[kMaxD];
#pragma unroll
      for (int j = kMaxD - 1; j >= 0; --j) stride[j] = (j >= m - 1) ? 1 : stride[j + 1 < kMaxD ? j + 1 : j] * z.v[j + 1 < kMaxD ? j + 1 : j];
      if (m == 3) {
        // two other modes u < v: the parts split over both, v fastest, and walk
        // them without divisions
        const int u = f == 0 ? 1 : 0, v = f == 2 ? 1 : 2;
        int sf = 1, su = 1, sv = 1, zu = 1, zv = 1;
#pragma unroll
        for (int j = 0; j < kMaxD; ++j) {
          if (j == f) sf = stride[j];
          if (j == u) { su = stride[j]; zu = z.v[j]; }
          if (j == v) { sv = stride[j]; zv = z.v[j]; }
        }
        const int nv = min(nparts, zv), nu = nparts / nv;
        const int pv = pp % nv, pu = pp / nv;
        if (pu < nu)
          for (int iu = pu; iu < zu; iu += nu) {
            const T mu = mv[u][iu];
            const T* Zr = Zl + a * sf + iu * su;
            for (int iv = pv; iv < zv; iv += nv) acc += Zr[iv * sv] * (mv[v][iv] * mu);
          }
      } else {
        int sf = 1;
#pragma unroll
        for (int j = 0; j < kMaxD; ++j)
          if (j == f) sf = stride[j];
        for (int o = pp; o < O; o += nparts) {
          int rem = o, row = a * sf;
          T prod = T(1);
#pragma unroll
          for (int j = kMaxD - 1; j >= 0; --j) {
            if (j >= m || j == f) continue;
            const int ij = rem % z.v[j];
            rem /= z.v[j];
            row += ij * stride[j];
            prod *= mv[j][ij];
          }
          acc += Zl[row] * prod;
        }
      }
    }
    part[tid] = acc;
    __syncthreads();
    if (tid < zf) {
      T s = T(0);
      for (int q = 0; q < nparts; ++q) s += part[q * zf + tid];
      T* o = tk_.out + tid + (size_t)l * ldo;
      const T v = T(coef) * s;
      *o = tk_.accumulate ? *o + v : v;
    }
  } else {
    T acc = T(0);
    for (int e = tid; e < P; e += KRP_NT) {
      int rem = e;
      T prod = T(1);
#pragma unroll
      for (int j = kMaxD - 1; j >= 0; --j) {
        if (j >= m) continue;
        const int ij = rem % z.v[j];
        rem /= z.v[j];
        prod *= mv[j][ij];
      }
      acc += Zl[e] * prod;
    }
    __shared__ T red[KRP_NT / kWave];
    const T s = block_sum(acc, red);
    if (tid == 0) {
      T* o = tk_.out + (size_t)l * ldo;
      const T v = T(coef) * s;
      *o = tk_.accumulate ? *o + v : v;
    }
  }
}

// Dot products, `parts` workgroups each; 16-byte loads, eight in flight per
// thread.  One CU reads about 50 GB/s, so a long product is spread: workgroup c
// of a product takes the elements [c, c + 1) * chunk and leaves a partial sum
// that dot_sum_kernel adds in order.
template <typename T> struct Vec16;
template <> struct Vec16<float> { typedef float V __attribute__((ext_vector_type(4))); static constexpr int W = 4; };
template <> struct Vec16<double> { typedef double V __attribute__((ext_vector_type(2))); static constexpr int W = 2; };

template <typename T>
__device__ __forceinline__ double vdot(const typename Vec16<T>::V& a, const typename Vec16<T>::V& b);
template <>
__device__ __forceinline__ double vdot<float>(const Vec16<float>::V& a, const Vec16<float>::V& b) {
  return double(a.x) * double(b.x) + double(a.y) * double(b.y) + double(a.z) * double(b.z) + double(a.w) * double(b.w);
}
template <>
__device__ __forceinline__ double vdot<double>(const Vec16<double>::V& a, const Vec16<double>::V& b) {
  return a.x * b.x + a.y * b.y;
}

constexpr int DOT_NT = 1024;

template <typename T>
__global__ __launch_bounds__(DOT_NT) void dot_kernel(const T* const* xs, const T* const* ys, size_t len, size_t chunk,
                                                     double scale, double* out) {
  __shared__ double red[DOT_NT / kWave];
  using V = typename Vec16<T>::V;
  constexpr int W = Vec16<T>::W;
  const size_t at = blockIdx.x * chunk;
  const T* x = xs[blockIdx.y] + at;
  const T* y = ys[blockIdx.y] + at;
  const size_t n = min(chunk, len - at);
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  size_t head = 0;
  if (((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y)) & 15) == 0) {
    const GPtr<V> xv = (GPtr<V>)x;
    const GPtr<V> yv = (GPtr<V>)y;
    const size_t nv = n / W;
    size_t e = threadIdx.x;
    if (x == y) {  // a squared norm reads its array once
      for (; e + 7 * DOT_NT < nv; e += 8 * DOT_NT) {
        V v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = xv[e + u * DOT_NT];
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u & 3] += vdot<T>(v[u], v[u]);
      }
    }
    for (; e + 3 * DOT_NT < nv; e += 4 * DOT_NT) {
      V v[4], w[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = xv[e + u * DOT_NT];
#pragma unroll
      for (int u = 0; u < 4; ++u) w[u] = yv[e + u * DOT_NT];
#pragma unroll
      for (int u = 0; u < 4; ++u) a[u] += vdot<T>(v[u], w[u]);
    }
    for (; e < nv; e += DOT_NT) {
      const V v = xv[e], w = yv[e];
      a[0] += vdot<T>(v, w);
    }
    head = nv * W;
  }
  for (size_t e = head + threadIdx.x; e < n; e += DOT_NT) a[1] += double(x[e]) * double(y[e]);
  const double sum = block_sum((a[0] + a[1]) + (a[2] + a[3]), red);
  if (threadIdx.x == 0) out[blockIdx.y * gridDim.x + blockIdx.x] = scale * sum;
}

// Adds the partial sums of one product, up to kDotParts of them, in order of a
// tree over the lanes.
__global__ __launch_bounds__(kWave) void dot_sum_kernel(const double* part, int parts, double scale, double* out) {
  const int l = threadIdx.x;
  const double v = wave_sum(l < parts ? part[size_t(blockIdx.x) * parts + l] : 0.0);
  if (l == 0) out[blockIdx.x] = scale * v;
}

template <typename T>
__global__ void scale_kernel(const T* __restrict__ x, T* __restrict__ y, size_t len, double scale, const double* num,
                             const double* den) {
  double a = scale;
  if (num) a *= *num;
  if (den) {
    // a norm as denominator: zero (a breakdown) or non-finite gives a zero
    // result instead of inf / NaN
    const double dv = *den;
    a = (dv > 0.0 && dv < INFINITY) ? a / dv : 0.0;
  }
  const T at = T(a);
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < len; e += (size_t)gridDim.x * blockDim.x)
    y[e] = at * x[e];
}

template <typename T>
__global__ void fill_kernel(T* y, size_t len, T v) {
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < len; e += (size_t)gridDim.x * blockDim.x)
    y[e] = v;
}

// Counts the non-finite entries of every task's array into *count (zeroed by
// the caller); one atomic per non-finite entry found.
__global__ void nonfinite_kernel(const double* const* xs, const size_t* lens, int ntasks, int* count) {
  const int t = blockIdx.y;
  if (t >= ntasks) return;
  const double* x = xs[t];
  const size_t len = lens[t];
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < len; e += (size_t)gridDim.x * blockDim.x)
    if (!isfinite(x[e])) atomicAdd(count, 1);
}

template <typename A, typename B>
__global__ void cast_kernel(const A* __restrict__ x, B* __restrict__ y, size_t len) {
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < len; e += (size_t)gridDim.x * blockDim.x)
    y[e] = B(x[e]);
}

template <typename A, typename B>
__global__ void cast_multi_kernel(CastSet<A, B> set) {
  const A* x = nullptr;
  B* y = nullptr;
  size_t len = 0;
#pragma unroll
  for (int k = 0; k < kMaxD; ++k)
    if (k == int(blockIdx.y)) {
      x = set.x[k];
      y = set.y[k];
      len = set.len[k];
    }
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < len; e += (size_t)gridDim.x * blockDim.x)
    y[e] = B(x[e]);
}

// dst (dims dd, row-major, `total` elements) = the indices of src (dims sd)
// below sv, zero outside.  I is unsigned where `total` fits in it (a 64-bit
// remainder costs several times a 32-bit one).
template <typename I, typename S, typename D>
__device__ __forceinline__ void recap_loop(GPtr<S> src, D* dst, I total, int d, const int* dd, const int* sd,
                                           const int* sv, I e0, I step) {
  for (I e = e0; e < total; e += step) {
    I rem = e;
    size_t so = 0, sstr = 1;
    bool inside = true;
#pragma unroll
    for (int k = kMaxD - 1; k >= 0; --k) {
      if (k >= d) continue;
      const int ik = int(rem % I(dd[k]));
      rem /= I(dd[k]);
      inside = inside && ik < sv[k] && ik < sd[k];
      so += size_t(ik) * sstr;
      sstr *= size_t(sd[k]);
    }
    dst[e] = inside ? D(src[so]) : D(0);
  }
}

template <typename S, typename D>
__device__ __forceinline__ void recap(GPtr<S> src, D* dst, size_t total, int d, const int* dd, const int* sd,
                                      const int* sv) {
  const unsigned e0 = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
  if (total <= 0x7fffffffu)
    recap_loop<unsigned>(src, dst, unsigned(total), d, dd, sd, sv, e0, step);
  else
    recap_loop<size_t>(src, dst, total, d, dd, sd, sv, size_t(e0), size_t(step));
}

template <typename S, typename D>
__device__ __forceinline__ void move_one(const MoveTask<S, D>& t) {
  const size_t e0 = size_t(blockIdx.x) * blockDim.x + threadIdx.x, step = size_t(gridDim.x) * blockDim.x;
  if (t.rank != nullptr && e0 < kMaxD) t.rank[e0] = t.rk[e0];
  const GPtr<S> src = (GPtr<S>)t.src;
  if (t.d == 0) {
    for (size_t e = e0; e < t.total; e += step) t.dst[e] = e < t.valid ? D(src[e]) : D(0);
  } else {
    recap(src, t.dst, t.total, t.d, t.dd, t.sd, t.sv);
  }
}

// Latency: a part is 1 to 24 KB per block at working sizes, so what counts is
// that all parts of all blocks go in one launch (three rank-48 blocks at
// n = 512: 15 launches and three rank copies, 36 us, before).
template <typename S, typename D>
__global__ __launch_bounds__(256) void move_parts_kernel(const MoveTask<S, D>* __restrict__ tasks) {
  const MoveTask<S, D> t = tasks[blockIdx.y];
  move_one(t);
}

template <typename S, typename D>
__global__ __launch_bounds__(256) void move_set_kernel(MoveSet<S, D> set) {
#pragma unroll
  for (int i = 0; i < kMoveSet; ++i)
    if (i == int(blockIdx.y)) move_one(set.t[i]);
}

// Ranks are read on the device, so the copies do not wait for a round trip of
// the ranks through the host: one launch, one copy back and one wait in place
// of d + 1 launches, two copies and two waits.
template <typename T>
__global__ __launch_bounds__(256) void export_kernel(ExportArgs<T> a) {
  int r[kMaxD], sd[kMaxD];
  bool fits = true;
#pragma unroll
  for (int k = 0; k < kMaxD; ++k) {
    r[k] = k < a.d ? a.rank[k] : 1;
    sd[k] = a.rc;
    if (k < a.d) fits = fits && r[k] >= 1 && r[k] <= a.rcap[k];
  }
  if (blockIdx.y == 0 && blockIdx.x == 0 && threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < kMaxD; ++k) a.hdr[k] = k < a.d ? r[k] : 0;
    a.hdr[kMaxD] = a.s_dev ? *a.s_dev : 0;
  }
  if (!fits) return;
  if (blockIdx.y == 0) {
    size_t total = 1;
#pragma unroll
    for (int k = 0; k < kMaxD; ++k) total *= k < a.d ? size_t(a.rcap[k]) : size_t(1);
    recap<T, double>((GPtr<T>)a.core, a.out_core, total, a.d, a.rcap, sd, r);
    return;
  }
  const size_t e0 = size_t(blockIdx.x) * blockDim.x + threadIdx.x, step = size_t(gridDim.x) * blockDim.x;
#pragma unroll
  for (int k = 0; k < kMaxD; ++k)
    if (k + 1 == int(blockIdx.y)) {
      const GPtr<T> src = (GPtr<T>)a.U[k];
      const size_t total = size_t(a.n[k]) * size_t(a.rcap[k]);
      const size_t valid = size_t(a.n[k]) * size_t(min(r[k], a.rc));
      for (size_t e = e0; e < total; e += step) a.out_U[k][e] = e < valid ? double(src[e]) : 0.0;
    }
}

template <typename T>
__global__ void core_recap_kernel(const T* __restrict__ src, Dims4 sd, Dims4 sv, T* __restrict__ dst, Dims4 dd,
                                  int d, size_t total) {
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
    size_t rem = e, so = 0, sstr = 1;
    bool inside = true;
    for (int k = d - 1; k >= 0; --k) {
      const int ik = int(rem % dd.v[k]);
      rem /= dd.v[k];
      if (ik >= sv.v[k] || ik >= sd.v[k]) inside = false;
      so += size_t(ik) * sstr;
      sstr *= sd.v[k];
    }
    dst[e] = inside ? src[so] : T(0);
  }
}

// core_recap_kernel without a view limit, and the zero-sum fix-up of the
// same step: when *tot <= *zthr (or NaN) the core is zero, every factor is
// e_1 in its first column and every rank is 1.
template <typename T>
__global__ void core_recap_fixup_kernel(const T* __restrict__ src, Dims4 sd, T* __restrict__ dst, Dims4 dd, int d,
                                        size_t total, const double* tot, const double* zthr, Dims4 nn, int rc,
                                        T* U0, T* U1, T* U2, T* U3, int* rank) {
  const bool zs = !(*tot > *zthr);
  const size_t tid = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  const size_t nth = (size_t)gridDim.x * blockDim.x;
  for (size_t e = tid; e < total; e += nth) {
    size_t rem = e, so = 0, sstr = 1;
    bool inside = true;
    for (int k = d - 1; k >= 0; --k) {
      const int ik = int(rem % dd.v[k]);
      rem /= dd.v[k];
      if (ik >= sd.v[k]) inside = false;
      so += size_t(ik) * sstr;
      sstr *= sd.v[k];
    }
    dst[e] = (inside && !zs) ? src[so] : T(0);
  }
  if (!zs) return;
  T* Us[4] = {U0, U1, U2, U3};
  for (int k = 0; k < d; ++k) {
    const size_t len = size_t(nn.v[k]) * rc;
    for (size_t e = tid; e < len; e += nth) Us[k][e] = (e == 0) ? T(1) : T(0);
  }
  if (tid < size_t(d)) rank[tid] = 1;
}

template <typename T>
__global__ void mat_recap_kernel(const T* __restrict__ src, int lds, int rs, int cs, T* __restrict__ dst, int ldd,
                                 int rd, int cd) {
  const size_t total = size_t(rd) * cd;
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
    const int i = int(e % rd), j = int(e / rd);
    dst[i + size_t(j) * ldd] = (i < rs && j < cs) ? src[i + size_t(j) * lds] : T(0);
  }
}

__global__ void sketch_width_kernel(const int* rt, int d, int p, int cap, int force, int* s_out) {
  if (threadIdx.x != 0) return;
  if (force >= 0) {
    *s_out = force;
    return;
  }
  int est = 0;
  for (int k = 0; k < d; ++k) {
    const int v = rt[k] < 0 ? cap + p : rt[k] + p;
    est = v > est ? v : est;
  }
  *s_out = est < cap + p ? est : cap + p;
}

__global__ void gram_prep_kernel(const int* const* ranks, int nb, int d, int rmax, int rreg, double* enable, int* nact,
                                 int* skip_small, int* skip_big) {
  const int k = threadIdx.x;
  if (k >= d) return;
  int R = 0;
  for (int b = 0; b < nb; ++b) R += ranks[b][k];
  enable[k] = R <= rmax ? 1.0 : 0.0;
  nact[k] = R <= rmax ? R : -1;
  skip_small[k] = R > rreg;
  skip_big[k] = R <= rreg;
}

// Compacts the lower triangle of a padded block Gram: compact index i maps to
// (block b, local a) through the prefix sums of the block ranks.
template <typename T>
__global__ void gram_compact_kernel(const T* __restrict__ padded, int ldp, const int* const* ranks, int nb, int rc,
                                    const int* nact, T* __restrict__ compact, int ldc, size_t msp, size_t msc) {
  const int k = blockIdx.y;
  const int R = nact[k];
  if (R <= 0) return;
  const T* P = padded + k * msp;
  T* C = compact + k * msc;
  const size_t total = size_t(R) * R;
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
    const int i = int(e % R), j = int(e / R);
    if (i < j) continue;
    int bi = 0, oi = i;
    while (oi >= ranks[bi][k]) { oi -= ranks[bi][k]; ++bi; }
    int bj = 0, oj = j;
    while (oj >= ranks[bj][k]) { oj -= ranks[bj][k]; ++bj; }
    C[i + size_t(j) * ldc] = P[(bi * rc + oi) + size_t(bj * rc + oj) * ldp];
  }
}

inline unsigned grid_for(size_t n, unsigned nt = 256) {
  size_t g = (n + nt - 1) / nt;
  return (unsigned)(g < 2048 ? (g == 0 ? 1 : g) : 2048);
}

}  // namespace

template <typename T>
void krp_reduce(const KrpTask<T>* tasks_d, int ntasks, int m, const int* z, int P, int S, hipStream_t st) {
  if (ntasks <= 0 || S <= 0) return;
  Dims4 zz{};
  for (int j = 0; j < m; ++j) {
    zz.v[j] = z[j];
    TK_CHECK(z[j] <= KRP_ZMAX, kErrUnsupported, "Khatri-Rao reduction: mode size above 128");
  }
  timer_begin(kKcKrp, st);
  hipLaunchKernelGGL((krp_kernel<T>), dim3(S, ntasks), dim3(KRP_NT), 0, st, tasks_d, m, zz, P, S);
  TK_LAUNCH_CHECK();
  timer_end(kKcKrp, st);
}

// A second launch costs 4 us and more, a single workgroup 1 us per 8 K
// elements (FP64): spread from 64 K elements on (three squared norms of 110 K
// elements 16.6 us in one workgroup each, FP64; one of 1.9 M elements 216 us).
int dot_parts(size_t len) {
  if (len < 65536) return 1;
  return int(std::min<size_t>(kDotParts, len / 8192));
}

template <typename T>
void dot_batched(const T* const* xs, const T* const* ys, size_t len, int n, double scale, double* out, double* part,
                 hipStream_t st) {
  if (n <= 0) return;
  const int parts = part != nullptr ? dot_parts(len) : 1;
  const size_t chunk = ((len + parts - 1) / parts + 3) / 4 * 4;  // keeps the 16-byte alignment
  hipLaunchKernelGGL((dot_kernel<T>), dim3(parts, n), dim3(DOT_NT), 0, st, xs, ys, len, parts == 1 ? len : chunk,
                     parts == 1 ? scale : 1.0, parts == 1 ? out : part);
  TK_LAUNCH_CHECK();
  if (parts > 1) {
    hipLaunchKernelGGL(dot_sum_kernel, dim3(n), dim3(kWave), 0, st, part, parts, scale, out);
    TK_LAUNCH_CHECK();
  }
}

template <typename T>
void scale_copy(const T* x, T* y, size_t len, double scale, const double* num, const double* den, hipStream_t st) {
  hipLaunchKernelGGL((scale_kernel<T>), dim3(grid_for(len)), dim3(256), 0, st, x, y, len, scale, num, den);
  TK_LAUNCH_CHECK();
}

void count_nonfinite(const double* const* xs, const size_t* lens, int ntasks, size_t maxlen, int* count,
                     hipStream_t st) {
  if (ntasks <= 0) return;
  hipLaunchKernelGGL(fill_kernel<int>, dim3(1), dim3(64), 0, st, count, size_t(1), 0);
  TK_LAUNCH_CHECK();
  hipLaunchKernelGGL(nonfinite_kernel, dim3(std::min<unsigned>(grid_for(maxlen), 256u), ntasks), dim3(256), 0, st, xs,
                     lens, ntasks, count);
  TK_LAUNCH_CHECK();
}

template <typename T>
void fill(T* y, size_t len, T v, hipStream_t st) {
  if (len == 0) return;
  hipLaunchKernelGGL((fill_kernel<T>), dim3(grid_for(len)), dim3(256), 0, st, y, len, v);
  TK_LAUNCH_CHECK();
}

template <typename A, typename B>
void cast_multi(const CastSet<A, B>& set, hipStream_t st) {
  TK_CHECK(set.count >= 0 && set.count <= kMaxD, kErrInvalidArg, "cast_multi: too many buffers");
  size_t mx = 0;
  for (int k = 0; k < set.count; ++k) mx = std::max(mx, set.len[k]);
  if (mx == 0) return;
  hipLaunchKernelGGL((cast_multi_kernel<A, B>), dim3(grid_for(mx), set.count), dim3(256), 0, st, set);
  TK_LAUNCH_CHECK();
}

template <typename A, typename B>
void cast_copy(const A* x, B* y, size_t len, hipStream_t st) {
  if (len == 0) return;
  hipLaunchKernelGGL((cast_kernel<A, B>), dim3(grid_for(len)), dim3(256), 0, st, x, y, len);
  TK_LAUNCH_CHECK();
}

template <typename S, typename D>
void move_parts(const MoveTask<S, D>* tasks_d, int ntasks, size_t maxtotal, hipStream_t st) {
  if (ntasks <= 0 || maxtotal == 0) return;
  const unsigned gx = unsigned(std::min<size_t>((maxtotal + 1023) / 1024, 512));  // about 4 elements a thread
  hipLaunchKernelGGL((move_parts_kernel<S, D>), dim3(gx, ntasks), dim3(256), 0, st, tasks_d);
  TK_LAUNCH_CHECK();
}

template <typename S, typename D>
void move_set(const MoveSet<S, D>& set, hipStream_t st) {
  TK_CHECK(set.count >= 1 && set.count <= kMoveSet, kErrInvalidArg, "move_set: number of parts");
  size_t mx = 1;
  for (int i = 0; i < set.count; ++i) mx = std::max<size_t>(mx, set.t[i].total);
  const unsigned gx = unsigned(std::min<size_t>((mx + 1023) / 1024, 512));
  hipLaunchKernelGGL((move_set_kernel<S, D>), dim3(gx, set.count), dim3(256), 0, st, set);
  TK_LAUNCH_CHECK();
}

template <typename T>
void export_parts(const ExportArgs<T>& a, hipStream_t st) {
  size_t mx = 1, core = 1;
  for (int k = 0; k < a.d; ++k) {
    core *= size_t(a.rcap[k]);
    mx = std::max(mx, size_t(a.n[k]) * a.rcap[k]);
  }
  mx = std::max(mx, core);
  const unsigned gx = unsigned(std::min<size_t>((mx + 1023) / 1024, 512));
  hipLaunchKernelGGL((export_kernel<T>), dim3(gx, a.d + 1), dim3(256), 0, st, a);
  TK_LAUNCH_CHECK();
}

template <typename T>
void core_recap(const T* src, const int* sd, const int* sv, T* dst, const int* dd, int d, hipStream_t st) {
  Dims4 a{}, v{}, b{};
  size_t total = 1;
  for (int k = 0; k < d; ++k) {
    a.v[k] = sd[k];
    v.v[k] = sv ? sv[k] : sd[k];
    b.v[k] = dd[k];
    total *= size_t(dd[k]);
  }
  hipLaunchKernelGGL((core_recap_kernel<T>), dim3(grid_for(total)), dim3(256), 0, st, src, a, v, dst, b, d, total);
  TK_LAUNCH_CHECK();
}

template <typename T>
void core_recap_fixup(const T* src, const int* sd, T* dst, const int* dd, int d, const double* total,
                      const double* zthr, const int* n, int rc, T* const* U, int* rank, hipStream_t st) {
  Dims4 a{}, b{}, nn{};
  T* uu[4] = {nullptr, nullptr, nullptr, nullptr};
  size_t len = 1, mx = 1;
  for (int k = 0; k < d; ++k) {
    a.v[k] = sd[k];
    b.v[k] = dd[k];
    nn.v[k] = n[k];
    uu[k] = U[k];
    len *= size_t(dd[k]);
    mx = std::max(mx, size_t(n[k]) * rc);
  }
  hipLaunchKernelGGL((core_recap_fixup_kernel<T>), dim3(grid_for(std::max(len, mx))), dim3(256), 0, st, src, a, dst,
                     b, d, len, total, zthr, nn, rc, uu[0], uu[1], uu[2], uu[3], rank);
  TK_LAUNCH_CHECK();
}

template <typename T>
void mat_recap(const T* src, int ld_src, int rows_src, int cols_src, T* dst, int ld_dst, int rows_dst, int cols_dst,
               hipStream_t st) {
  const size_t total = size_t(rows_dst) * cols_dst;
  if (total == 0) return;
  hipLaunchKernelGGL((mat_recap_kernel<T>), dim3(grid_for(total)), dim3(256), 0, st, src, ld_src, rows_src, cols_src,
                     dst, ld_dst, rows_dst, cols_dst);
  TK_LAUNCH_CHECK();
}

void gram_prep(const int* const* ranks, int nb, int d, int rmax, int rreg, double* enable, int* nact, int* skip_small,
               int* skip_big, hipStream_t st) {
  hipLaunchKernelGGL(gram_prep_kernel, dim3(1), dim3(64), 0, st, ranks, nb, d, rmax, rreg, enable, nact, skip_small,
                     skip_big);
  TK_LAUNCH_CHECK();
}

template <typename T>
void gram_compact(const T* padded, int ldp, const int* const* ranks, int nb, int d, int rc, const int* nact,
                  T* compact, int ldc, size_t mode_stride_p, size_t mode_stride_c, hipStream_t st) {
  hipLaunchKernelGGL((gram_compact_kernel<T>), dim3(64, d), dim3(256), 0, st, padded, ldp, ranks, nb, rc, nact,
                     compact, ldc, mode_stride_p, mode_stride_c);
  TK_LAUNCH_CHECK();
}

void sketch_width(const int* rt, int d, int p, int cap, int force, int* s_out, hipStream_t st) {
  hipLaunchKernelGGL(sketch_width_kernel, dim3(1), dim3(64), 0, st, rt, d, p, cap, force, s_out);
  TK_LAUNCH_CHECK();
}

#define TK_INST(T)                                                                                         \
  template void krp_reduce<T>(const KrpTask<T>*, int, int, const int*, int, int, hipStream_t);             \
  template void dot_batched<T>(const T* const*, const T* const*, size_t, int, double, double*, double*, hipStream_t); \
  template void scale_copy<T>(const T*, T*, size_t, double, const double*, const double*, hipStream_t);    \
  template void fill<T>(T*, size_t, T, hipStream_t);                                                       \
  template void core_recap<T>(const T*, const int*, const int*, T*, const int*, int, hipStream_t);         \
  template void mat_recap<T>(const T*, int, int, int, T*, int, int, int, hipStream_t);                     \
  template void core_recap_fixup<T>(const T*, const int*, T*, const int*, int, const double*, const double*,    \
                                    const int*, int, T* const*, int*, hipStream_t);                     \
  template void gram_compact<T>(const T*, int, const int* const*, int, int, int, const int*, T*, int, size_t, \
                                size_t, hipStream_t);
TK_INST(double)
TK_INST(float)
#undef TK_INST
template void move_parts<double, double>(const MoveTask<double, double>*, int, size_t, hipStream_t);
template void move_parts<double, float>(const MoveTask<double, float>*, int, size_t, hipStream_t);
template void move_parts<float, double>(const MoveTask<float, double>*, int, size_t, hipStream_t);
template void move_set<double, double>(const MoveSet<double, double>&, hipStream_t);
template void export_parts<double>(const ExportArgs<double>&, hipStream_t);
template void export_parts<float>(const ExportArgs<float>&, hipStream_t);
template void cast_copy<double, float>(const double*, float*, size_t, hipStream_t);
template void cast_multi<double, float>(const CastSet<double, float>&, hipStream_t);
template void cast_multi<float, double>(const CastSet<float, double>&, hipStream_t);
template void cast_copy<float, double>(const float*, double*, size_t, hipStream_t);
template void fill<int>(int*, size_t, int, hipStream_t);

}  // namespace tk
