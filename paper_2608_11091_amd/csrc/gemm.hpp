// Grouped, batched GEMM on CDNA4 matrix cores.
//
// One launch computes, for every group g,
//     C_g = beta * C_g + sum_{t in terms(g)} alpha_t * op(A_t) * op(B_t)
// with column-major operands, of uniform shape M x N x K unless the launch is
// mixed.  alpha_t is
// scale_t * (*c1_t) * (*c2_t) with optional device scalars, so
// device-resident coefficients (inner products, least-squares solutions,
// block weights) scale terms without a host round trip.  Term and group
// tables live in device memory and are built once per plan.
#pragma once

#include "common.hpp"

namespace tk {

template <typename T>
struct GemmTerm {
  const T* A;
  const T* B;
  const double* c1;  // optional device scalar (nullptr = 1)
  const double* c2;  // optional device scalar (nullptr = 1)
  const double* gate;  // read when the launch is gated: 0 leaves the term out
  double scale;
};

template <typename T>
struct GemmGroup {
  T* C;
  int t0, t1;  // term range [t0, t1)
  int M, K, lda, ldb, ldc;  // read when the launch is mixed
  int ops;                  // transposes, read when the launch has any_ops: op(A) = A^T (1), op(B) = B^T (2)
};

// Launch descriptor: uniform transposes and N, device tables.
template <typename T>
struct GemmLaunch {
  bool ta = false, tb = false;
  bool any_ops = false;    // transposes per group (tile 32)
  int M = 0, N = 0, K = 0, lda = 0, ldb = 0, ldc = 0;
  const GemmTerm<T>* terms = nullptr;   // device
  const GemmGroup<T>* groups = nullptr; // device
  int ngroups = 0;
  double beta = 0.0;
  int tile = 64;           // side of a workgroup's output tile: 64 or 32
  int splits = 1;          // split of the (term x K-slab) space (>1 uses `partial` + a reduction pass)
  T* partial = nullptr;    // ngroups * splits * M * N
  T* folded = nullptr;     // folds > 0: the deferred partials are first summed into folds of them here
  int folds = 0;           // (ngroups * folds * M * N)
  int uniform_terms = 0;   // > 0: group g has the terms [g u, (g + 1) u)
  bool mixed = false;      // groups have their own M, K, lda, ldb, ldc (M, K above: the largest)
  // mblk > 0 (A not transposed): row i of A and C is row i % mblk of slice
  // i / mblk, the slices astr and cstr elements apart (a product over a middle
  // mode of a tensor, whose slices would each fill their tiles in part)
  int mblk = 0;
  long astr = 0, cstr = 0;
  int max_terms = 1 << 30; // clamp every group to its first max_terms terms
  bool gated = false;      // groups of one term, left out (C = 0) where its gate is 0
  bool bf16 = false;       // FP32 storage: round the operands to bfloat16, BF16 matrix cores, FP32 accumulation
  bool defer_reduce = false;  // splits > 1: leave the partials for the consumer to sum (C is not written)
  double flops = 0.0;      // algorithmic flops of this launch (for the kernel timer)
};

template <typename T>
void gemm_run(const GemmLaunch<T>& g, hipStream_t st);

}  // namespace tk
