// Grouped GEMM kernel on MFMA (v_mfma_f64_16x16x4f64 / v_mfma_f32_16x16x4f32).
//
// Tile: 64 x 64 outputs per workgroup of 256 threads (4 waves), or 32 x 32 where
// that leaves most of the chip idle.  In the large tile a wave owns a strip of
// 16 rows or 16 columns and up to four MFMA 16 x 16 accumulators along it; the
// strips run along the shorter live side, so a product with 15, 32 or 37
// columns issues 1, 2 or 3 MFMAs a step in place of 4 (FP64 16x16x4: 64 cycles
// each on its SIMD).  In the small tile a wave owns one accumulator.  K is
// staged through LDS in slabs of 32 (large tile), 64 (small tile) or 16 (bf16
// form), eight loads per operand and thread, coalesced along the contiguous
// dimension of each operand; halves of a slab and k steps beyond the operands
// are neither loaded nor multiplied, and the alpha of a term is folded into the
// A slab while it is staged.  A small launch is bound by its chain of
// latencies (table, operands, LDS, MFMAs, store): the small tile has a quarter
// of the MFMAs of a wave and one slab where the large one has two.
#include "gemm.hpp"

#include <type_traits>

#include "kernels.hpp"

namespace tk {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

template <typename T> struct Acc;
template <> struct Acc<double> { typedef d4 type; static constexpr bool f64 = true; };
template <> struct Acc<float> { typedef f4 type; static constexpr bool f64 = false; };

__device__ __forceinline__ d4 mfma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// BF16 operand form (FP32 storage and accumulation): operands are rounded to
// bfloat16 (round to nearest even; NaN kept quiet) as they are staged, and
// multiplied on v_mfma_f32_16x16x16_bf16.  Lane l supplies rows / columns
// l % 16 and the four consecutive k values 4 (l / 16) .. 4 (l / 16) + 3.
typedef short s4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ unsigned short bf16_rne(float x) {
  unsigned u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ f4 mfma_bf16(s4 a, s4 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

constexpr int NT = 256;

// Rows in slices (GemmLaunch::mblk); the quotient by a multiplication, exact
// while rows * mblk < 2^32.
struct RowBlocks {
  unsigned mblk, magic;
  long astr, cstr;
  __device__ __forceinline__ size_t at(int row, long str) const {
    if (mblk == 0) return size_t(row);
    const unsigned s = __umulhi(unsigned(row), magic);
    return size_t(s) * size_t(str) + (unsigned(row) - s * mblk);
  }
};

// Whether a value that is the same in every lane is zero, as a scalar condition.
__device__ __forceinline__ bool uniform_zero(float x) {
  return (__builtin_amdgcn_readfirstlane(__float_as_int(x)) & 0x7fffffff) == 0;
}
__device__ __forceinline__ bool uniform_zero(double x) {
  const int lo = __builtin_amdgcn_readfirstlane(__double2loint(x));
  const int hi = __builtin_amdgcn_readfirstlane(__double2hiint(x));
  return (lo | (hi & 0x7fffffff)) == 0;
}

// Split-K: the (term, K-slab) iteration space of a group is divided evenly
// over `splits` workgroups per output tile; each writes its partial tile and a
// second pass sums the partials in split order.  (Summing them in the last
// workgroup to arrive at a tile needs device-scope fences, whose L2
// write-back across the XCDs cost more than the second launch.)
// OPS: bit 0 op(A) = A^T, bit 1 op(B) = B^T; kAnyOps: as each group says.
constexpr int kAnyOps = 4;
template <typename T, int OPS, int TS, bool BF = false>
__global__ __launch_bounds__(NT) void gemm_kernel(int M, int N, int K, int lda, int ldb, int ldc,
                                                  const GemmTerm<T>* __restrict__ terms,
                                                  const GemmGroup<T>* __restrict__ groups, double beta,
                                                  int splits, T* __restrict__ partial, size_t pstride,
                                                  int max_terms, int uniform_terms, bool mixed, bool gated,
                                                  RowBlocks rb_) {
  static_assert(!BF || sizeof(T) == 4, "bf16 operands with FP32 storage only");
  static_assert(!BF || TS == 64, "bf16 operands with the large tile only");
  static_assert(OPS != kAnyOps || TS == 32, "operations per group with the small tile only");
  // K depth of a slab: 8 loads per operand and thread in flight at once (16
  // for the bf16 form, one 16-deep MFMA per output tile)
  constexpr int BM = TS, BN = TS, KB = BF ? 16 : TS == 64 ? 32 : 64;
  constexpr int SA = (BM * KB) / NT, SB = (BN * KB) / NT;  // staged elements per thread
  constexpr int NACC = TS == 64 ? 4 : 1;
  constexpr int BKP = 16 + 4;  // bf16 row: 16 k values + 4 pad (40 bytes: conflict-free 8-byte reads)
  static_assert(BM == BN, "one row length for both slabs");
  __shared__ T slabs[2][BF ? 1 : KB][BM + 1];  // [A, B][k][m or n]
  auto& As = slabs[0];
  auto& Bs = slabs[1];
  __shared__ __align__(8) unsigned short Asb[BF ? BM : 1][BKP];  // [m][k]
  __shared__ __align__(8) unsigned short Bsb[BF ? BN : 1][BKP];  // [n][k]
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
  const int g = blockIdx.z / splits;
  const int sp = blockIdx.z % splits;
  // A launch of uniform groups knows its term range from the arguments, so the
  // first term's record is not behind the group's.
  const GemmGroup<T> grp = groups[g];
  int t0 = g * uniform_terms, t1 = t0 + uniform_terms;
  if (uniform_terms == 0) {
    t0 = grp.t0;
    t1 = grp.t1;
  }
  if (mixed) {
    M = grp.M;
    K = grp.K;
    lda = grp.lda;
    ldb = grp.ldb;
    ldc = grp.ldc;
    if (m0 >= M) return;
  }
  const int ops = OPS == kAnyOps ? grp.ops : OPS;
  const bool TA = ops & 1, TB = ops & 2;

  typedef typename Acc<T>::type AT;
  AT acc[NACC];
#pragma unroll
  for (int i = 0; i < NACC; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[i][v] = T(0);

  const int nterm = max(0, min(t1 - t0, max_terms));
  const int nks = (K + KB - 1) / KB;
  const int total = nterm * nks;
  const int per = (total + splits - 1) / splits;
  const int sb = sp * per;
  int se = min(total, sb + per);
  // a term that is left out is not read (its alpha is known only after its
  // operands are on their way)
  if (gated && nterm > 0 && uniform_zero(*terms[t0].gate)) se = sb;
  const int Ml = min(BM, M - m0), Nl = min(BN, N - n0);  // live rows and columns of the tile
  const int mt = (Ml + 15) >> 4, nt = (Nl + 15) >> 4;
  // large tile: a wave owns 16 rows (or 16 columns) of it and `live`
  // accumulators; small tile: one of its 2 x 2 accumulators
  const bool by_rows = nt < mt;
  const int wi = wid & 1, wj = wid >> 1;
  const int live = TS == 32 ? (wi < mt && wj < nt ? 1 : 0) : by_rows ? (wid < mt ? nt : 0) : (wid < nt ? mt : 0);

  // staging coordinates of this thread (fixed over slabs): element i of A is
  // row am0 + i * amd, k ak0 + i * akd of the slab
  const int tm0 = tid % TS, tk0 = TS == 64 ? wid : tid / TS;
  const int am0 = TA ? tid / KB : tm0, ak0 = TA ? tid % KB : tk0;
  const int amd = TA ? NT / KB : 0, akd = TA ? 0 : NT / TS;
  const int bn0 = TB ? tm0 : tid / KB, bk0 = TB ? tk0 : tid % KB;
  const int bnd = TB ? 0 : NT / KB, bkd = TB ? NT / TS : 0;
  // Slab s is fetched into registers one slab ahead of its use, so its global
  // loads are in flight while the matrix cores work on slab s - 1; the record
  // of the next term is fetched one term ahead, and a term's coefficients are
  // first needed when its slab is staged.  The loads are unconditional up to
  // halves of the slab (indices clamp to the operand) and go through the
  // global address space; k steps beyond the operand become zeros and the
  // term's alpha is applied when the slab is staged into LDS: a select or a
  // multiply right after a load, or a flat load (counted with the LDS
  // operations that every barrier waits for), would make the thread wait for
  // that load before issuing the next.  Rows and columns beyond the operands
  // hold copies of the last one (or what the LDS held): they only reach
  // accumulators that are not stored.  A term with alpha == 0 is not
  // multiplied, whatever its operands hold.
  int t = t0, kf = 0;  // term and k of the slab to fetch
  GemmTerm<T> tm = {}, tn = {};
  double c1 = 1.0, c2 = 1.0, sc = 0.0;  // coefficients of the fetched slab's term
  T ra[SA], rb[SB];
  auto coefs = [&]() {
    sc = tm.scale;
    c1 = tm.c1 ? *tm.c1 : 1.0;
    c2 = tm.c2 ? *tm.c2 : 1.0;
  };
  const size_t arow = TA ? 0 : rb_.at(min(m0 + am0, M - 1), rb_.astr);  // (one row per thread when A is not transposed)
  auto load = [&]() {
    const GPtr<T> ga = (GPtr<T>)tm.A;
    const GPtr<T> gb = (GPtr<T>)tm.B;
    const bool a2 = SA / 2 * amd < Ml && kf + SA / 2 * akd < K, b2 = SB / 2 * bnd < Nl && kf + SB / 2 * bkd < K;
    auto la = [&](int i) {
      const int gk = min(kf + ak0 + i * akd, K - 1);
      ra[i] = TA ? ga[gk + (size_t)min(m0 + am0 + i * amd, M - 1) * lda] : ga[arow + (size_t)gk * lda];
    };
    auto lb = [&](int i) {
      const int gn = min(n0 + bn0 + i * bnd, N - 1), gk = min(kf + bk0 + i * bkd, K - 1);
      rb[i] = TB ? gb[gn + (size_t)gk * ldb] : gb[gk + (size_t)gn * ldb];
    };
#pragma unroll
    for (int i = 0; i < SA / 2; ++i) la(i);
#pragma unroll
    for (int i = 0; i < SB / 2; ++i) lb(i);
    if (a2)
#pragma unroll
      for (int i = SA / 2; i < SA; ++i) la(i);
    if (b2)
#pragma unroll
      for (int i = SB / 2; i < SB; ++i) lb(i);
  };
  if (sb < se) {
    t = t0 + sb / nks;
    kf = (sb - (t - t0) * nks) * KB;
    tm = terms[t];
    if (t + 1 < t0 + nterm) tn = terms[t + 1];
    load();
    coefs();
  }
  T alpha = T(0);
  int ks = 0;  // k of the slab being staged
  bool fresh = true;  // its term's coefficients have not been multiplied yet
  for (int slab = sb; slab < se; ++slab) {
    ks = kf;
    if (fresh) {
      double al = sc;
      al *= c1;
      al *= c2;
      alpha = T(al);
    }
    auto next = [&]() {  // fetch the following slab
      fresh = false;
      if (slab + 1 >= se) return;
      kf += KB;
      if (kf >= K) {
        kf = 0;
        ++t;
        tm = tn;
        if (t + 1 < t0 + nterm) tn = terms[t + 1];
        fresh = true;
      }
      load();
      if (fresh) coefs();
    };
    // a slab of a zero-coefficient term adds nothing: it is neither staged nor
    // multiplied
    if (uniform_zero(alpha)) {
      next();
      continue;
    }
    const int kl = K - ks;  // live k of the slab
    if constexpr (BF) {
#pragma unroll
      for (int i = 0; i < SA; ++i)
        Asb[am0 + i * amd][ak0 + i * akd] =
            bf16_rne(float(ak0 + i * akd < kl ? ra[i] * alpha : T(0)));
#pragma unroll
      for (int i = 0; i < SB; ++i)
        Bsb[bn0 + i * bnd][bk0 + i * bkd] =
            bf16_rne(float(bk0 + i * bkd < kl ? rb[i] : T(0)));
    } else {
      auto sa = [&](int i) { As[ak0 + i * akd][am0 + i * amd] = ak0 + i * akd < kl ? ra[i] * alpha : T(0); };
      auto sb_ = [&](int i) { Bs[bk0 + i * bkd][bn0 + i * bnd] = bk0 + i * bkd < kl ? rb[i] : T(0); };
#pragma unroll
      for (int i = 0; i < SA / 2; ++i) sa(i);
#pragma unroll
      for (int i = 0; i < SB / 2; ++i) sb_(i);
      if (SA / 2 * amd < Ml && SA / 2 * akd < kl)
#pragma unroll
        for (int i = SA / 2; i < SA; ++i) sa(i);
      if (SB / 2 * bnd < Nl && SB / 2 * bkd < kl)
#pragma unroll
        for (int i = SB / 2; i < SB; ++i) sb_(i);
    }
    __syncthreads();
    next();
    if constexpr (BF) {
      // the whole 16-deep slab in one MFMA per 16 x 16 output tile
      const int kq = 4 * (lane >> 4), c = lane & 15;
      if (by_rows) {
        const s4 a = *reinterpret_cast<const s4*>(&Asb[wid * 16 + c][kq]);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (j < live) acc[j] = mfma_bf16(a, *reinterpret_cast<const s4*>(&Bsb[j * 16 + c][kq]), acc[j]);
      } else {
        const s4 b = *reinterpret_cast<const s4*>(&Bsb[wid * 16 + c][kq]);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (j < live) acc[j] = mfma_bf16(*reinterpret_cast<const s4*>(&Asb[j * 16 + c][kq]), b, acc[j]);
      }
    } else if constexpr (TS == 32) {
      if (live) {
#pragma unroll
        for (int k0 = 0; k0 < KB; k0 += 16) {
          if (k0 >= kl) continue;
          T x[4], y[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int kr = k0 + 4 * u + (lane >> 4), c = lane & 15;
            x[u] = As[kr][wi * 16 + c];
            y[u] = Bs[kr][wj * 16 + c];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) acc[0] = mfma(x[u], y[u], acc[0]);
        }
      }
    } else {
      // strip operand x (one 16-wide strip) against y (`live` strips)
      const auto& xs = slabs[by_rows ? 0 : 1];
      const auto& ys = slabs[by_rows ? 1 : 0];
      auto strips = [&](auto lv, auto rows) {
        constexpr int LV = decltype(lv)::value;
        auto half = [&](int k0) {
#pragma unroll
          for (int kk = 0; kk < 16; kk += 4) {
            const int kr = k0 + kk + (lane >> 4), c = lane & 15;
            const T x = xs[kr][wid * 16 + c];
            T y[LV];
#pragma unroll
            for (int j = 0; j < LV; ++j) y[j] = ys[kr][j * 16 + c];
#pragma unroll
            for (int j = 0; j < LV; ++j)
              acc[j] = decltype(rows)::value ? mfma(x, y[j], acc[j]) : mfma(y[j], x, acc[j]);
          }
        };
        half(0);
        if (kl > 16) half(16);
      };
      auto sized = [&](auto rows) {
        if (live == 4) strips(std::integral_constant<int, 4>{}, rows);
        else if (live == 3) strips(std::integral_constant<int, 3>{}, rows);
        else if (live == 2) strips(std::integral_constant<int, 2>{}, rows);
        else if (live == 1) strips(std::integral_constant<int, 1>{}, rows);
      };
      if (by_rows) sized(std::true_type{});
      else sized(std::false_type{});
    }
    __syncthreads();
  }

  // Accumulator layout of a 16x16 tile (measured on gfx950): for FP32, D[r][c]
  // sits in lane c + 16*(r/4), element r%4; for FP64 in lane c + 16*(r%4),
  // element r/4.
#pragma unroll
  for (int j = 0; j < NACC; ++j)
    if (j < live) {
      const int ti = TS == 32 ? wi : by_rows ? wid : j, tj = TS == 32 ? wj : by_rows ? j : wid;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r16 = Acc<T>::f64 ? 4 * v + (lane >> 4) : 4 * (lane >> 4) + v;
        const int row = m0 + ti * 16 + r16;
        const int col = n0 + tj * 16 + (lane & 15);
        if (row < M && col < N) {
          if (splits == 1) {
            T* c = grp.C + rb_.at(row, rb_.cstr) + (size_t)col * ldc;
            *c = (beta == 0.0) ? acc[j][v] : T(beta) * (*c) + acc[j][v];
          } else {
            partial[(size_t)blockIdx.z * pstride + (size_t)col * M + row] = acc[j][v];
          }
        }
      }
    }
}

// Sums the partials of every group into `folds` of them.  A chunk's partials are summed in order, 16 loads in flight.
template <typename T>
__global__ __launch_bounds__(256) void splitk_fold(size_t MN, int splits, int folds, const T* __restrict__ partial,
                                                   T* __restrict__ out) {
  const int per = (splits + folds - 1) / folds;
  const int s0 = blockIdx.y * per, s1 = min(splits, s0 + per);
  const size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (e >= MN) return;
  const GPtr<T> p = (GPtr<T>)(partial + (size_t)blockIdx.z * splits * MN + e);
  T a = T(0);
  for (int s = s0; s < s1; s += 16) {
    T v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = p[size_t(min(s + u, s1 - 1)) * MN];
#pragma unroll
    for (int u = 0; u < 16; ++u) a += s + u < s1 ? v[u] : T(0);
  }
  out[((size_t)blockIdx.z * folds + blockIdx.y) * MN + e] = a;
}

template <typename T>
__global__ void splitk_reduce(int M, int N, int ldc, const GemmGroup<T>* __restrict__ groups, double beta,
                              int splits, const T* __restrict__ partial, size_t pstride, bool mixed) {
  const int g = blockIdx.y;
  const GemmGroup<T> grp = groups[g];
  if (mixed) {
    M = grp.M;
    ldc = grp.ldc;
  }
  const unsigned MN = unsigned(M) * unsigned(N);
  for (unsigned e = blockIdx.x * blockDim.x + threadIdx.x; e < MN; e += gridDim.x * blockDim.x) {
    // eight loads in flight; the additions keep their order
    const GPtr<T> p = (GPtr<T>)(partial + (size_t)g * splits * pstride + e);
    T s = T(0);
    for (int sp = 0; sp < splits; sp += 8) {
      T v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p[(size_t)min(sp + u, splits - 1) * pstride];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += sp + u < splits ? v[u] : T(0);
    }
    const int row = int(e % unsigned(M)), col = int(e / unsigned(M));
    T* c = grp.C + row + (size_t)col * ldc;
    *c = (beta == 0.0) ? s : T(beta) * (*c) + s;
  }
}

}  // namespace

template <typename T>
void gemm_run(const GemmLaunch<T>& g, hipStream_t st) {
  if (g.ngroups <= 0 || g.M <= 0 || g.N <= 0) return;
  TK_CHECK(g.bf16 || g.any_ops ? g.tile == (g.bf16 ? 64 : 32) : g.tile == 64 || g.tile == 32, kErrInvalidArg,
           "internal: product tile");
  dim3 grid(ceil_div(g.M, g.tile), ceil_div(g.N, g.tile), g.ngroups * g.splits);
  T* part = g.splits > 1 ? g.partial : nullptr;
  const size_t pstride = (size_t)g.M * g.N;
  RowBlocks rb{};
  if (g.mblk > 0) {
    TK_CHECK(!g.ta && !g.any_ops && g.splits == 1 && !g.mixed && long(g.M) * g.mblk < (1L << 32), kErrInvalidArg,
             "internal: rows in slices");
    rb.mblk = unsigned(g.mblk);
    rb.magic = unsigned(((1ull << 32) + rb.mblk - 1) / rb.mblk);
    rb.astr = g.astr;
    rb.cstr = g.cstr;
  }
  timer_begin(kKcGemm, st, g.flops);
  TK_CHECK(!g.bf16 || sizeof(T) == 4, kErrUnsupported, "bf16 operands need FP32 storage");
  const int ops = g.any_ops ? kAnyOps : (g.ta ? 1 : 0) + (g.tb ? 2 : 0);
#define TK_GEMM_CASE(OPS, TS, BF)                                                                              \
  if (ops == OPS && g.tile == TS && g.bf16 == BF)                                                              \
    hipLaunchKernelGGL((gemm_kernel<T, OPS, TS, BF && sizeof(T) == 4>), grid, dim3(NT), 0, st, g.M, g.N, g.K,  \
                       g.lda, g.ldb, g.ldc, g.terms, g.groups, g.beta, g.splits, part, pstride, g.max_terms,   \
                       g.uniform_terms, g.mixed, g.gated, rb);
#define TK_GEMM_CASES(TS, BF)         \
  TK_GEMM_CASE(0, TS, BF)             \
  TK_GEMM_CASE(1, TS, BF)             \
  TK_GEMM_CASE(2, TS, BF)             \
  TK_GEMM_CASE(3, TS, BF)
  TK_GEMM_CASES(32, false)
  TK_GEMM_CASE(kAnyOps, 32, false)
  TK_GEMM_CASES(64, false)
  if constexpr (sizeof(T) == 4) {
    TK_GEMM_CASES(64, true)
  }
#undef TK_GEMM_CASES
#undef TK_GEMM_CASE
  TK_LAUNCH_CHECK();
  if (g.folds > 0) {
    TK_CHECK(g.defer_reduce && g.folded != nullptr && g.splits > 1 && g.ngroups <= 65535, kErrInvalidArg,
             "internal: folded partials need a deferred reduction");
    dim3 fg((unsigned)((pstride + 255) / 256), g.folds, g.ngroups);
    hipLaunchKernelGGL((splitk_fold<T>), fg, dim3(256), 0, st, pstride, g.splits, g.folds, part, g.folded);
    TK_LAUNCH_CHECK();
  }
  if (g.splits > 1 && !g.defer_reduce) {
    dim3 rg((unsigned)std::min<size_t>((pstride + 255) / 256, 64), g.ngroups);
    hipLaunchKernelGGL((splitk_reduce<T>), rg, dim3(256), 0, st, g.M, g.N, g.ldc, g.groups, g.beta, g.splits, part,
                       pstride, g.mixed);
    TK_LAUNCH_CHECK();
  }
  timer_end(kKcGemm, st);
}

template void gemm_run<double>(const GemmLaunch<double>&, hipStream_t);
template void gemm_run<float>(const GemmLaunch<float>&, hipStream_t);

}  // namespace tk
