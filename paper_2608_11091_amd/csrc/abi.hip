// C ABI of the library (declared in include/tsgmres.h): argument checks,
// import of caller tensors into capacity-padded internal layouts, planning
// (measure-only for the *_workspace queries), execution and export.
#include <algorithm>
#include <cmath>
#include <map>
#include <memory>
#include <mutex>

#include "../../include/tsgmres.h"
#include "engine.hpp"

namespace tk {

static thread_local std::string g_err;
const char* last_error() { return g_err.c_str(); }

template <typename F>
static int guarded(F&& f) {
  try {
    g_err.clear();
    return f();
  } catch (const Error& e) {
    g_err = e.msg;
    return e.code;
  } catch (const std::exception& e) {
    g_err = e.what();
    return kErrInvalidArg;
  } catch (...) {
    g_err = "unknown error";
    return kErrInvalidArg;
  }
}

namespace {

void check_tucker(const tk_tucker* t, const char* name, int d, const int64_t* n) {
  TK_CHECK(t != nullptr, kErrInvalidArg, std::string(name) + " is NULL");
  TK_CHECK(t->d == d, kErrShape, std::string(name) + ": order mismatch");
  TK_CHECK(t->core != nullptr, kErrInvalidArg, std::string(name) + ": core is NULL");
  for (int k = 0; k < d; ++k) {
    TK_CHECK(t->n[k] == n[k], kErrShape, std::string(name) + ": mode size mismatch");
    TK_CHECK(t->r[k] >= 1 && t->r[k] <= t->rcap[k], kErrShape, std::string(name) + ": rank outside [1, rcap]");
    TK_CHECK(t->r[k] <= t->n[k], kErrShape, std::string(name) + ": rank above mode size");
    TK_CHECK(t->U[k] != nullptr, kErrInvalidArg, std::string(name) + ": factor is NULL");
  }
}

void check_dims(int d, const int64_t* n) {
  TK_CHECK(d >= 2 && d <= kMaxD, kErrUnsupported, "order d must be in [2, 4]");
  for (int k = 0; k < d; ++k) {
    TK_CHECK(n[k] >= 1, kErrShape, "mode sizes must be positive");
    TK_CHECK(n[k] <= 512, kErrUnsupported, "mode sizes above 512 are not supported");
  }
}

void check_op(const tk_kron_op* op, int d, const int64_t* n) {
  TK_CHECK(op != nullptr, kErrInvalidArg, "operator is NULL");
  TK_CHECK(op->d == d, kErrShape, "operator order mismatch");
  for (int k = 0; k < d; ++k) TK_CHECK(op->n[k] == n[k], kErrShape, "operator mode size mismatch");
  TK_CHECK(op->nterms >= 1 && op->alpha != nullptr && op->A != nullptr, kErrInvalidArg, "operator has no terms");
}

// Whether a caller tensor's core (k < 0) or factor k already has the capacity
// layout: nothing to cut, pad or convert.
bool in_layout(const Shape& sh, const tk_tucker& u, int k) {
  if (k >= 0) return u.r[k] == sh.rc;
  for (int j = 0; j < sh.d; ++j)
    if (u.r[j] != sh.rc || u.rcap[j] != sh.rc) return false;
  return true;
}

// Arrays a call writes before its last read of the inputs.
using Writes = std::vector<std::pair<const double*, size_t>>;
bool overlaps(const Writes& w, const double* p, size_t len) {
  for (auto& x : w)
    if (x.first != nullptr && x.first < p + len && p < x.first + x.second) return true;
  return false;
}

// The moves that bring a caller tensor into the capacity layout: core,
// factors and ranks.  With `in_place` the parts that have the layout, and that
// none of those writes touches, are used where they are (the plan only reads
// them): t then points at them, and the move of such a part is empty (it keeps
// its place in the table, so that the workspace depends on capacities alone).
template <typename D>
void import_tasks(const Shape& sh, const tk_tucker& u, TT<D>& t, std::vector<MoveTask<double, D>>& out,
                  const Writes* in_place = nullptr) {
  const int d = sh.d;
  MoveTask<double, D> c{};
  c.src = u.core;
  c.dst = t.core;
  c.total = sh.core_len();
  c.d = d;
  c.rank = t.rank;
  bool inner = true;  // modes 1 .. d - 1 keep their strides: one contiguous piece
  size_t slice = 1;
  for (int k = 0; k < kMaxD; ++k) {
    c.sd[k] = k < d ? int(u.rcap[k]) : 1;
    c.sv[k] = k < d ? int(u.r[k]) : 1;
    c.dd[k] = k < d ? sh.rc : 1;
    c.rk[k] = k < d ? int(u.r[k]) : 1;
    if (k >= 1 && k < d) {
      inner &= u.r[k] == sh.rc && u.rcap[k] == sh.rc;
      slice *= size_t(sh.rc);
    }
  }
  if (inner) {  // no index arithmetic (it costs four times the copy of a large core)
    c.d = 0;
    c.valid = slice * size_t(u.r[0]);
  }
  if constexpr (std::is_same<D, double>::value)
    if (in_place && in_layout(sh, u, -1) && !overlaps(*in_place, u.core, sh.core_len())) {
      t.core = const_cast<double*>(u.core);
      c.total = c.valid = 0;
    }
  out.push_back(c);
  for (int k = 0; k < d; ++k) {
    MoveTask<double, D> f{};
    f.src = u.U[k];
    f.dst = t.U[k];
    f.total = size_t(sh.n[k]) * sh.rc;
    f.valid = size_t(sh.n[k]) * size_t(u.r[k]);
    if constexpr (std::is_same<D, double>::value)
      if (in_place && in_layout(sh, u, k) && !overlaps(*in_place, u.U[k], f.total)) {
        t.U[k] = const_cast<double*>(u.U[k]);
        f.total = f.valid = 0;
      }
    out.push_back(f);
  }
}

// A plain array converted from S to D.
template <typename S, typename D>
MoveTask<S, D> convert_task(const S* src, D* dst, size_t len) {
  MoveTask<S, D> t{};
  t.src = src;
  t.dst = dst;
  t.total = t.valid = len;
  return t;
}

// One launch for all moves of a call (the table goes into the plan's blob).
template <typename S, typename D>
void emit_moves(Seq& q, Planner& pl, const std::vector<MoveTask<S, D>>& tasks) {
  size_t mx = 1;
  for (auto& t : tasks) mx = std::max<size_t>(mx, t.total);
  const size_t off = pl.blob.add(tasks);
  const int nt = int(tasks.size());
  Blob* bl = &pl.blob;
  q.steps.push_back([=](hipStream_t st) { move_parts<S, D>(bl->at<MoveTask<S, D>>(off), nt, mx, st); });
}

// Import of one tensor outside a plan (tasks as kernel arguments).
void emit_import(Seq& q, const Shape& sh, const tk_tucker& u, TT<double> t) {
  std::vector<MoveTask<double, double>> tasks;
  import_tasks<double>(sh, u, t, tasks);
  MoveSet<double, double> set;
  for (auto& x : tasks) set.t[set.count++] = x;
  q.steps.push_back([=](hipStream_t st) { move_set<double, double>(set, st); });
}

constexpr int kExportHdr = kMaxD + 1;  // ints of the export's header

// Copies an internal tensor out and reads its ranks (and the width *s_dev)
// back; `hdr` holds kExportHdr device ints.
template <typename T>
void export_tt(const Shape& sh, const TT<T>& t, tk_tucker* u, int* hdr, const int* s_dev, int32_t* s_out,
               hipStream_t st) {
  ExportArgs<T> a{};
  a.core = t.core;
  a.rank = t.rank;
  a.s_dev = s_dev;
  a.out_core = u->core;
  a.d = sh.d;
  a.rc = sh.rc;
  a.hdr = hdr;
  for (int k = 0; k < sh.d; ++k) {
    a.U[k] = t.U[k];
    a.out_U[k] = u->U[k];
    a.n[k] = sh.n[k];
    a.rcap[k] = int(u->rcap[k]);
  }
  export_parts<T>(a, st);
  int h[kExportHdr] = {0};
  TK_HIP(hipMemcpyAsync(h, hdr, sizeof(h), hipMemcpyDeviceToHost, st));
  TK_HIP(hipStreamSynchronize(st));
  if (s_out) *s_out = h[kMaxD];
  for (int k = 0; k < sh.d; ++k)
    TK_CHECK(h[k] >= 1 && h[k] <= u->rcap[k], kErrCapacity,
             "output rank " + std::to_string(h[k]) + " exceeds the capacity of the output tensor");
  for (int k = 0; k < sh.d; ++k) u->r[k] = h[k];
}

void check_form(int form) {
  TK_CHECK(form == TK_FORM_FP64 || form == TK_FORM_FP32 || form == TK_FORM_BF16, kErrUnsupported, "unknown form");
}

void finish_blob(Arena& ar, Blob& blob, hipStream_t st) {
  blob.dev = ar.alloc<unsigned char>(std::max<size_t>(blob.host.size(), 16));
  if (!ar.measuring())
    TK_HIP(hipMemcpyAsync(blob.dev, blob.host.data(), blob.host.size(), hipMemcpyHostToDevice, st));
}

Shape shape_of(int d, const int64_t* n, int rc, int cap, int p) {
  Shape sh;
  sh.d = d;
  for (int k = 0; k < d; ++k) sh.n[k] = int(n[k]);
  sh.rc = rc;
  sh.cap = cap;
  sh.p = p;
  return sh;
}

// ---------------------------------------------------------------- apply
int do_apply(const tk_kron_op* op, const tk_tucker* x, int transpose, int form, double* const* AU, Arena& ar,
             hipStream_t st) {
  TK_CHECK(x != nullptr, kErrInvalidArg, "x is NULL");
  check_dims(x->d, x->n);
  check_op(op, x->d, x->n);
  check_tucker(x, "x", x->d, x->n);
  check_form(form);
  const int d = x->d;
  Blob blob;
  Planner pl(ar, blob);
  pl.bf16_factors = form == TK_FORM_BF16;
  const bool f32 = form != TK_FORM_FP64;  // FP32 storage (FP32 and BF16-factor forms)
  Seq q;
  // the products of one shape (mode size, rank capacity) share a launch
  struct Product {
    const double* A;
    double* out;
    int k;
  };
  std::map<std::pair<int, int>, std::vector<Product>> shapes;
  for (int j = 0; j < op->nterms; ++j)
    for (int k = 0; k < d; ++k) {
      const double* A = op->A[j * d + k];
      if (!A) continue;
      TK_CHECK(AU != nullptr && AU[j * d + k] != nullptr, kErrInvalidArg, "missing output buffer for a factor product");
      shapes[{int(x->n[k]), int(x->rcap[k])}].push_back(Product{A, AU[j * d + k], k});
    }
  // FP32 storage: operands rounded by one launch, results widened by one
  // (every product converts its own operand: the workspace does not depend on
  // which pointers coincide)
  std::vector<MoveTask<double, float>> down;
  std::vector<MoveTask<float, double>> up;
  auto f32_of = [&](const double* src, size_t len) {
    float* dst = ar.alloc<float>(len);
    down.push_back(convert_task<double, float>(src, dst, len));
    return static_cast<const float*>(dst);
  };
  std::array<const float*, kMaxD> U32{};
  if (f32)
    for (int k = 0; k < d; ++k) U32[k] = f32_of(x->U[k], size_t(x->n[k]) * x->rcap[k]);
  Seq prod;
  for (auto& sh : shapes) {
    const int n = sh.first.first, rcap = sh.first.second;
    const size_t len = size_t(n) * rcap;
    if (f32) {
      std::vector<const float*> a, b;
      std::vector<float*> c;
      for (auto& p : sh.second) {
        a.push_back(f32_of(p.A, size_t(n) * n));
        b.push_back(U32[p.k]);
        c.push_back(ar.alloc<float>(len));
        up.push_back(convert_task<float, double>(c.back(), p.out, len));
      }
      plan_gemm_batched<float>(prod, pl, !transpose, false, n, rcap, n, a, n, b, n, c, n, 1.0, true);
    } else {
      std::vector<const double*> a, b;
      std::vector<double*> c;
      for (auto& p : sh.second) {
        a.push_back(p.A);
        b.push_back(x->U[p.k]);
        c.push_back(p.out);
      }
      plan_gemm_batched<double>(prod, pl, !transpose, false, n, rcap, n, a, n, b, n, c, n, 1.0);
    }
  }
  if (f32) emit_moves(q, pl, down);
  for (auto& f : prod.steps) q.steps.push_back(f);
  if (f32) emit_moves(q, pl, up);
  finish_blob(ar, blob, st);
  if (ar.measuring()) return 0;
  q.run(st);
  TK_HIP(hipStreamSynchronize(st));
  return 0;
}

// Finiteness check of the inputs of a solve, run before any other kernel
// reads them: a non-finite entry makes the call fail with TK_ERR_NONFINITE.
// Tensors are checked after their import into the capacity layout, where the
// entries beyond the ranks are zero.
struct FiniteCheck {
  std::vector<const double*> ptr;
  std::vector<size_t> len;
  const double** dptr = nullptr;
  size_t* dlen = nullptr;
  int* count = nullptr;
  size_t room = 0;  // entries of the tables: null pointers count, as a query has no others
  void add(const double* p, size_t n) {
    ++room;
    if (p != nullptr && n > 0) {
      ptr.push_back(p);
      len.push_back(n);
    }
  }
  void add_tt(const Shape& sh, const TT<double>& t) {
    add(t.core, sh.core_len());
    for (int k = 0; k < sh.d; ++k) add(t.U[k], size_t(sh.n[k]) * sh.rc);
  }
  void add_inputs(const Shape& sh, const tk_kron_op* op, const double* const* S, int64_t s,
                  const double* const* omega, int wo, const tk_sgmres_params* prm) {
    const int d = sh.d;
    for (int j = 0; j < op->nterms; ++j)
      for (int k = 0; k < d; ++k) add(op->A[j * d + k], size_t(sh.n[k]) * sh.n[k]);
    for (int k = 0; k < d; ++k) {
      if (S) add(S[k], size_t(sh.n[k]) * size_t(s));
      add(omega[k], size_t(sh.n[k]) * size_t(wo));
      if (prm->precond_q > 0 && prm->precond_V && prm->precond_lambda) {
        add(prm->precond_V[k], size_t(sh.n[k]) * sh.n[k]);
        add(prm->precond_lambda[k], size_t(sh.n[k]));
      }
    }
  }
  void alloc(Arena& ar) {
    dptr = ar.alloc<const double*>(std::max<size_t>(room, 1));
    dlen = ar.alloc<size_t>(std::max<size_t>(room, 1));
    count = ar.alloc<int>(1);
  }
  void run(hipStream_t st) const {
    if (ptr.empty()) return;
    TK_HIP(hipMemcpyAsync(dptr, ptr.data(), sizeof(const double*) * ptr.size(), hipMemcpyHostToDevice, st));
    TK_HIP(hipMemcpyAsync(dlen, len.data(), sizeof(size_t) * len.size(), hipMemcpyHostToDevice, st));
    size_t mx = 0;
    for (size_t l : len) mx = std::max(mx, l);
    count_nonfinite(dptr, dlen, int(ptr.size()), mx, count, st);
    int h = 0;
    TK_HIP(hipMemcpyAsync(&h, count, sizeof(int), hipMemcpyDeviceToHost, st));
    TK_HIP(hipStreamSynchronize(st));
    TK_CHECK(h == 0, kErrNonFinite,
             std::to_string(h) + " non-finite input entries (right-hand side, initial guess, operator, sketches "
                                 "or preconditioner)");
  }
};

// ---------------------------------------------------------------- block sums
template <typename T>
struct Imported {
  Shape sh;
  Blocks<T> blocks;
};

// Shape of a block sum (checked), without importing it.
Shape shape_of_blocks(const tk_block_sum* in, int cap, int p) {
  TK_CHECK(in != nullptr && in->nblocks >= 1 && in->blocks != nullptr && in->coef != nullptr, kErrInvalidArg,
           "empty block sum");
  const tk_tucker& b0 = in->blocks[0];
  check_dims(b0.d, b0.n);
  int rc = std::max(cap, 1);
  for (int b = 0; b < in->nblocks; ++b) {
    check_tucker(&in->blocks[b], "block", b0.d, b0.n);
    for (int k = 0; k < b0.d; ++k) rc = std::max<int>(rc, int(in->blocks[b].r[k]));
  }
  TK_CHECK(rc <= 128, kErrUnsupported, "ranks above 128 are not supported");
  return shape_of(b0.d, b0.n, rc, cap, p);
}

// The blocks in the capacity layout, rounded to T; the moves are added to
// `tasks` (launched by the caller together with its own).  FP64 parts that
// have the layout are read where they are (`writes`: see import_tasks); their space stays reserved, so the
// workspace depends on the capacities alone.
template <typename T>
Imported<T> import_blocks(Arena& ar, const tk_block_sum* in, const Shape& sh, std::vector<MoveTask<double, T>>& tasks,
                          const Writes& writes = {}) {
  Imported<T> im;
  im.sh = sh;
  for (int b = 0; b < in->nblocks; ++b) {
    TT<T> t = alloc_tt<T>(ar, sh);
    import_tasks<T>(sh, in->blocks[b], t, tasks, &writes);
    im.blocks.add(t, nullptr, in->coef[b]);
  }
  return im;
}

// Sketch factors (n_k x w) rounded to FP32.
std::array<const float*, kMaxD> sketch_f32(Arena& ar, const Shape& sh, const double* const* S, size_t w,
                                           std::vector<MoveTask<double, float>>& tasks) {
  std::array<const float*, kMaxD> o{};
  for (int k = 0; k < sh.d; ++k) {
    float* dst = ar.alloc<float>(size_t(sh.n[k]) * w);
    tasks.push_back(convert_task<double, float>(S[k], dst, size_t(sh.n[k]) * w));
    o[k] = dst;
  }
  return o;
}

int do_sketch(const tk_block_sum* x, const double* const* S, int64_t s, int form, double* out, Arena& ar,
              hipStream_t st, bool lean = false) {
  TK_CHECK(S != nullptr && out != nullptr, kErrInvalidArg, "sketch factors or output missing");
  TK_CHECK(s >= 1 && s <= 65535, kErrInvalidArg, "sketch size out of range");
  check_form(form);
  Blob blob;
  Planner pl(ar, blob);
  Seq q;
  const Shape sh = shape_of_blocks(x, 1, 0);
  std::array<const double*, kMaxD> Sk{};
  for (int k = 0; k < sh.d; ++k) {
    TK_CHECK(S[k] != nullptr, kErrInvalidArg, "sketch factor is NULL");
    Sk[k] = S[k];
  }
  pl.bf16_factors = form == TK_FORM_BF16;
  pl.lean = lean;
  if (form != TK_FORM_FP64) {
    std::vector<MoveTask<double, float>> mv;
    const auto S32 = sketch_f32(ar, sh, Sk.data(), size_t(s), mv);
    const auto im = import_blocks<float>(ar, x, sh, mv);
    emit_moves(q, pl, mv);
    plan_sketch<float>(q, pl, sh, im.blocks, S32, int(s), out);
  } else if (lean) {  // one import launch per block, without a table
    Blocks<double> blocks;
    for (int b = 0; b < x->nblocks; ++b) {
      TT<double> t;  // (a sketch reads no ranks)
      t.core = ar.alloc<double>(sh.core_len());
      for (int k = 0; k < sh.d; ++k) t.U[k] = ar.alloc<double>(size_t(sh.n[k]) * sh.rc);
      emit_import(q, sh, x->blocks[b], t);
      blocks.add(t, nullptr, x->coef[b]);
    }
    plan_sketch<double>(q, pl, sh, blocks, Sk, int(s), out);
  } else {
    std::vector<MoveTask<double, double>> mv;
    const auto im = import_blocks<double>(ar, x, sh, mv);
    emit_moves(q, pl, mv);
    plan_sketch<double>(q, pl, sh, im.blocks, Sk, int(s), out);
  }
  finish_blob(ar, blob, st);
  if (ar.measuring()) return 0;
  q.run(st);
  TK_HIP(hipStreamSynchronize(st));
  return 0;
}

int do_rhosvd(const tk_block_sum* in, const tk_round_params* prm, const double* const* omega, tk_tucker* out,
              int32_t* s_out, Arena& ar, hipStream_t st) {
  TK_CHECK(prm != nullptr, kErrInvalidArg, "parameters are NULL");
  TK_CHECK(prm->rank_cap >= 1 && prm->oversample >= 0, kErrInvalidArg, "invalid rank cap / oversampling");
  TK_CHECK(prm->rank_cap + prm->oversample <= 64, kErrUnsupported, "rank_cap + oversample above 64");
  TK_CHECK(prm->eps >= 0.0, kErrInvalidArg, "eps must be >= 0");
  Blob blob;
  Planner pl(ar, blob);
  Seq q;
  const Shape sh = shape_of_blocks(in, prm->rank_cap, prm->oversample);
  TK_CHECK(prm->force_s < 0 || (prm->force_s >= 1 && prm->force_s <= sh.sc()), kErrInvalidArg,
           "force_s outside [1, rank_cap + oversample]");
  RoundCfg cfg;
  cfg.eps = prm->eps;
  cfg.tau = prm->tau;
  cfg.force_s = prm->force_s;
  for (int k = 0; k < sh.d; ++k) {
    cfg.force_r[k] = prm->force_ranks[k];
    TK_CHECK(cfg.force_r[k] <= prm->rank_cap, kErrInvalidArg, "forced rank above rank_cap");
  }
  std::array<const double*, kMaxD> om{};
  TK_CHECK(omega != nullptr, kErrInvalidArg, "omega is NULL");
  for (int k = 0; k < sh.d; ++k) om[k] = omega[k];
  if (out) check_dims(out->d, out->n);
  check_form(prm->form);
  TT<double> o;
  TT<float> o32;
  int* s_dev = nullptr;
  int* hdr = ar.alloc<int>(kExportHdr);
  const bool f32 = prm->form != TK_FORM_FP64;
  pl.bf16_factors = prm->form == TK_FORM_BF16;
  if (f32) {
    std::vector<MoveTask<double, float>> mv;
    const auto om32 = sketch_f32(ar, sh, om.data(), size_t(sh.sc()), mv);
    const auto im = import_blocks<float>(ar, in, sh, mv);
    emit_moves(q, pl, mv);
    o32 = alloc_tt<float>(ar, sh);
    s_dev = plan_roundsum<float>(q, pl, sh, im.blocks, cfg, om32, o32, nullptr).s_dev;
  } else {
    std::vector<MoveTask<double, double>> mv;
    const auto im = import_blocks<double>(ar, in, sh, mv);
    emit_moves(q, pl, mv);
    o = alloc_tt<double>(ar, sh);
    s_dev = plan_roundsum<double>(q, pl, sh, im.blocks, cfg, om, o, nullptr).s_dev;
  }
  finish_blob(ar, blob, st);
  if (ar.measuring()) return 0;
  TK_CHECK(out != nullptr && out->d == sh.d, kErrInvalidArg, "output tensor missing or of wrong order");
  for (int k = 0; k < sh.d; ++k) TK_CHECK(out->n[k] == sh.n[k], kErrShape, "output mode size mismatch");
  q.run(st);
  if (f32)
    export_tt<float>(sh, o32, out, hdr, s_dev, s_out, st);
  else
    export_tt<double>(sh, o, out, hdr, s_dev, s_out, st);
  return 0;
}

// Plans the exact norm of a block sum; returns where it leaves the square.
double* plan_norm(const tk_block_sum* x, const Shape& sh, bool share, Seq& q, Blob& blob, Arena& ar, hipStream_t st) {
  Planner pl(ar, blob);
  std::vector<MoveTask<double, double>> mv;
  const auto im = import_blocks<double>(ar, x, sh, mv);
  emit_moves(q, pl, mv);
  double* n2 = ar.alloc<double>(1);
  plan_exact_norm2(q, pl, im.sh, im.blocks, n2, share);
  finish_blob(ar, blob, st);
  return n2;
}

// The workspace is that of distinct factors: it must not depend on which
// pointers coincide, as the query may be asked with other ones.  Blocks that
// do share a factor are planned with it taken once where that plan fits in
// (it needs less but for its splits, which follow its own sizes).
int do_norm(const tk_block_sum* x, double* out, Arena& ar, hipStream_t st) {
  const Shape sh = shape_of_blocks(x, 1, 0);
  TK_CHECK(sh.rc <= 64, kErrUnsupported, "exact norm: ranks above 64");
  bool share = false;
  for (int k = 0; k < sh.d; ++k) {
    std::vector<const double*> u;
    for (int b = 0; b < x->nblocks; ++b) u.push_back(x->blocks[b].U[k]);
    std::sort(u.begin(), u.end());
    share |= std::adjacent_find(u.begin(), u.end()) != u.end();
  }
  Blob blob;
  Seq q;
  double* n2 = nullptr;
  if (share && !ar.measuring()) {
    size_t need[2] = {0, 0};  // of distinct, of shared factors
    for (int i = 0; i < 2; ++i) {
      Arena probe(nullptr, 0);
      Blob b;
      Seq s;
      plan_norm(x, sh, i == 1, s, b, probe, st);
      need[i] = probe.used();
    }
    TK_CHECK(ar.capacity() >= need[0], kErrWorkspace,
             "workspace too small: need at least " + std::to_string(need[0]) + " bytes");
    share = need[1] <= need[0];
  }
  n2 = plan_norm(x, sh, share && !ar.measuring(), q, blob, ar, st);
  if (ar.measuring()) return 0;
  TK_CHECK(out != nullptr, kErrInvalidArg, "output pointer is NULL");
  q.run(st);
  double h = 0.0;
  TK_HIP(hipMemcpyAsync(&h, n2, sizeof(double), hipMemcpyDeviceToHost, st));
  TK_HIP(hipStreamSynchronize(st));
  *out = std::sqrt(std::max(h, 0.0));
  return 0;
}

// ---------------------------------------------------------------- solve
SolveCfg solve_cfg(const tk_sgmres_params* prm) {
  SolveCfg c;
  c.form = prm->form;
  c.tol = prm->tol;
  c.eta = prm->eta;
  c.maxiter = prm->maxiter;
  c.max_restarts = prm->max_restarts;
  c.k_trunc = prm->k_trunc;
  c.s = int(prm->s);
  c.eps_trunc = prm->eps_trunc;
  c.eps_min = prm->eps_min;
  c.tol_inner_floor = prm->tol_inner_floor;
  c.tikhonov = prm->tikhonov != 0;
  c.method = prm->method;
  return c;
}

void check_params(const tk_sgmres_params* prm) {
  TK_CHECK(prm != nullptr, kErrInvalidArg, "parameters are NULL");
  TK_CHECK(prm->form == TK_FORM_FP64 || prm->form == TK_FORM_FP32, kErrUnsupported, "unknown precision form");
  TK_CHECK(prm->tol > 0 && prm->eta > 0 && prm->eta <= 1, kErrInvalidArg, "tol > 0 and 0 < eta <= 1 required");
  TK_CHECK(prm->maxiter >= 1 && prm->maxiter <= 64, kErrUnsupported, "maxiter must be in [1, 64]");
  TK_CHECK(prm->max_restarts >= 0, kErrInvalidArg, "max_restarts must be >= 0");
  TK_CHECK(prm->k_trunc >= 1, kErrInvalidArg, "k_trunc must be >= 1");
  TK_CHECK(prm->rank_cap >= 1 && prm->oversample >= 0 && prm->rank_cap + prm->oversample <= 64, kErrUnsupported,
           "rank_cap + oversample must be in [1, 64]");
  TK_CHECK(prm->method == 0 || prm->method == 1, kErrInvalidArg, "method must be 0 (sGMRES) or 1 (GMRES)");
  TK_CHECK(prm->method == 1 || (prm->s >= prm->maxiter && prm->s <= 256), kErrUnsupported,
           "sketch size must be in [maxiter, 256]");
  TK_CHECK(prm->method == 0 || prm->precond_q == 0, kErrUnsupported,
           "the preconditioner runs with the sketched cycles only (method 0)");
  TK_CHECK(prm->precond_q >= 0 && prm->precond_q <= 400, kErrInvalidArg, "precond_q must be in [0, 400]");
  TK_CHECK(prm->precond_q == 0 || (prm->precond_V != nullptr && prm->precond_lambda != nullptr), kErrInvalidArg,
           "preconditioner eigenpairs missing");
  TK_CHECK(prm->tikhonov == 0 || prm->tikhonov == 1, kErrInvalidArg, "tikhonov must be 0 or 1");
}

PrecondT<double> precond_of(const tk_sgmres_params* prm, int d) {
  PrecondT<double> pc;
  pc.q = prm->precond_q;
  if (pc.q > 0)
    for (int k = 0; k < d; ++k) {
      pc.V[k] = prm->precond_V[k];
      pc.lam[k] = prm->precond_lambda[k];
    }
  return pc;
}

OpDev<double> op_dev(const tk_kron_op* op) {
  OpDev<double> o;
  o.nterms = op->nterms;
  o.alpha.assign(op->alpha, op->alpha + op->nterms);
  for (int i = 0; i < op->nterms * op->d; ++i) o.A.push_back(op->A[i]);
  return o;
}

void fill_info(const SolveInfo& si, tk_sgmres_info* info, int d) {
  if (!info) return;
  info->status = si.status;
  info->iters_total = si.iters;
  info->cycles = si.cycles;
  info->true_relres = si.true_relres;
  info->seconds = si.seconds;
  const int nh = int(si.hist_sketched.size());
  info->hist_len = std::min(nh, std::max(0, info->hist_cap));
  for (int i = 0; i < info->hist_len; ++i) {
    if (info->hist_sketched) info->hist_sketched[i] = si.hist_sketched[i];
    if (info->hist_ranks)
      for (int k = 0; k < TK_MAX_D; ++k) info->hist_ranks[i * TK_MAX_D + k] = k < d ? si.hist_ranks[i * d + k] : 0;
  }
  if (info->hist_true)
    for (int i = 0; i < std::min<int>(int(si.hist_true.size()), info->hist_cap); ++i) info->hist_true[i] = si.hist_true[i];
  if (info->hist_cycle_seconds)
    for (int i = 0; i < std::min<int>(int(si.hist_time.size()), info->hist_cap); ++i)
      info->hist_cycle_seconds[i] = si.hist_time[i];
  if (info->hist_lambda)
    for (int i = 0; i < info->hist_cap; ++i)
      info->hist_lambda[i] = i < int(si.hist_lambda.size()) ? si.hist_lambda[i] : 0.0;
}

int do_solve(const tk_kron_op* op, const tk_tucker* b, const tk_sgmres_params* prm, const double* const* S,
             const double* const* omega, tk_tucker* x, tk_sgmres_info* info, Arena& ar, hipStream_t st) {
  TK_CHECK(b != nullptr, kErrInvalidArg, "b is NULL");
  check_dims(b->d, b->n);
  check_op(op, b->d, b->n);
  check_tucker(b, "b", b->d, b->n);
  check_params(prm);
  TK_CHECK((S != nullptr || prm->method == 1) && omega != nullptr, kErrInvalidArg, "sketch matrices missing");
  const int d = b->d;
  int rc = prm->rank_cap;
  for (int k = 0; k < d; ++k) rc = std::max<int>(rc, int(b->r[k]));
  if (prm->x0) {
    check_tucker(prm->x0, "x0", d, b->n);
    for (int k = 0; k < d; ++k) rc = std::max<int>(rc, int(prm->x0->r[k]));
  }
  TK_CHECK(rc <= 64, kErrUnsupported, "ranks above 64 are not supported by the solver");
  Shape sh = shape_of(d, b->n, rc, prm->rank_cap, prm->oversample);
  Seq imp;
  TT<double> bi = alloc_tt<double>(ar, sh);
  emit_import(imp, sh, *b, bi);
  TT<double> x0i;
  if (prm->x0) {
    x0i = alloc_tt<double>(ar, sh);
    emit_import(imp, sh, *prm->x0, x0i);
  }
  std::array<const double*, kMaxD> Sk{}, Ok{};
  for (int k = 0; k < d; ++k) {
    Sk[k] = S ? S[k] : nullptr;
    Ok[k] = omega[k];
  }
  auto solver = make_solver(ar, sh, op_dev(op), bi, solve_cfg(prm), Sk, Ok, prm->x0 ? &x0i : nullptr, st,
                            precond_of(prm, d));
  int* hdr = ar.alloc<int>(kExportHdr);
  FiniteCheck fin;
  fin.add_tt(sh, bi);
  if (prm->x0) fin.add_tt(sh, x0i);
  fin.add_inputs(sh, op, S, prm->s, omega, sh.sc(), prm);
  fin.alloc(ar);
  if (ar.measuring()) return 0;
  TK_CHECK(x != nullptr, kErrInvalidArg, "x is NULL");
  imp.run(st);
  fin.run(st);
  TT<double> xo;
  SolveInfo si;
  solver_run(*solver, xo, si, st);
  export_tt<double>(sh, xo, x, hdr, nullptr, nullptr, st);
  fill_info(si, info, d);
  return si.status;
}

// ---------------------------------------------------------------- backward
int do_backward(const tk_kron_op* op, const tk_tucker* x, const tk_block_sum* xbar, const tk_sgmres_params* prm,
                const double* const* S, const double* const* omega, tk_tucker* lambda, double* dalpha,
                double* const* dA, tk_sgmres_info* info, Arena& ar, hipStream_t st) {
  TK_CHECK(x != nullptr, kErrInvalidArg, "x is NULL");
  check_dims(x->d, x->n);
  check_op(op, x->d, x->n);
  check_tucker(x, "x", x->d, x->n);
  TK_CHECK(prm == nullptr || prm->tikhonov == 0, kErrUnsupported,
           "the adjoint gradients assume an unregularised solve (tikhonov must be 0)");
  TK_CHECK(prm == nullptr || prm->method == 0, kErrUnsupported, "the adjoint solve runs sGMRES cycles (method 0)");
  check_params(prm);
  TK_CHECK(S != nullptr && omega != nullptr, kErrInvalidArg, "sketch matrices missing");
  const int d = x->d;
  int rc = prm->rank_cap;
  for (int k = 0; k < d; ++k) rc = std::max<int>(rc, int(x->r[k]));
  TK_CHECK(xbar != nullptr && xbar->nblocks >= 1, kErrInvalidArg, "cotangent is empty");
  for (int b = 0; b < xbar->nblocks; ++b) {
    check_tucker(&xbar->blocks[b], "xbar block", d, x->n);
    for (int k = 0; k < d; ++k) rc = std::max<int>(rc, int(xbar->blocks[b].r[k]));
  }
  TK_CHECK(rc <= 64, kErrUnsupported, "ranks above 64 are not supported by the solver");
  Shape sh = shape_of(d, x->n, rc, prm->rank_cap, prm->oversample);
  Blob blob;
  Planner pl(ar, blob);
  Seq imp, pre, post;
  // import x and the cotangent blocks, round the cotangent (FP64)
  TT<double> xi = alloc_tt<double>(ar, sh);
  emit_import(imp, sh, *x, xi);
  FiniteCheck fin;
  fin.add_tt(sh, xi);
  Blocks<double> xb;
  for (int b = 0; b < xbar->nblocks; ++b) {
    TT<double> t = alloc_tt<double>(ar, sh);
    emit_import(imp, sh, xbar->blocks[b], t);
    fin.add_tt(sh, t);
    TK_CHECK(std::isfinite(xbar->coef[b]), kErrNonFinite, "cotangent coefficient is not finite");
    xb.add(t, nullptr, xbar->coef[b]);
  }
  std::array<const double*, kMaxD> Sk{}, Ok{};
  for (int k = 0; k < d; ++k) {
    Sk[k] = S[k];
    Ok[k] = omega[k];
  }
  RoundCfg rc_cfg;
  rc_cfg.eps = 1e-2 * prm->tol;
  TT<double> xbr = alloc_tt<double>(ar, sh);
  plan_roundsum<double>(pre, pl, sh, xb, rc_cfg, Ok, xbr, nullptr);
  // adjoint solve L^T lambda = xbar
  SolveCfg scfg = solve_cfg(prm);
  scfg.transpose = true;
  OpDev<double> od = op_dev(op);
  auto solver = make_solver(ar, sh, od, xbr, scfg, Sk, Ok, nullptr, st, precond_of(prm, d));
  // gradient contractions, planned for every solution slot of the solver
  double* dal = ar.alloc<double>(op->nterms);
  int* hdr = ar.alloc<int>(kExportHdr);
  Seq grad[3];
  for (int slot = 0; slot < 3; ++slot) {
    const TT<double> lam = solver_slot(*solver, slot);
    Seq& q = grad[slot];
    Blocks<double> lx = plan_apply<double>(q, pl, sh, od, xi, false);
    std::vector<double*> P;  // P[j*d+l] = U_lam,l^T A_j^(l) U_x,l
    plan_inner<double>(q, pl, sh, {lam}, lx, dal, -1.0, &P);
    if (dA == nullptr) continue;
    for (int j = 0; j < op->nterms; ++j)
      for (int k = 0; k < d; ++k) {
        if (op->A[j * d + k] == nullptr || dA[j * d + k] == nullptr) continue;
        int dims[kMaxD];
        for (int l = 0; l < d; ++l) dims[l] = sh.rc;
        const double* cur = xi.core;
        double* tA = ar.alloc<double>(sh.core_len());
        double* tB = ar.alloc<double>(sh.core_len());
        double* tgt = tA;
        for (int l = d - 1; l >= 0; --l) {
          if (l == k) continue;
          plan_ttm<double>(q, pl, d, dims, l, sh.rc, cur, P[j * d + l], sh.rc, false, tgt);
          cur = tgt;
          tgt = (tgt == tA) ? tB : tA;
        }
        double* Mid = ar.alloc<double>(size_t(sh.rc) * sh.rc);
        plan_unfold_gram<double>(q, pl, d, dims, k, lam.core, cur, Mid, sh.rc, 1.0);
        const int n = sh.n[k];
        double* tmp = ar.alloc<double>(size_t(n) * sh.rc);
        plan_gemm<double>(q, pl, false, true, n, sh.rc, sh.rc, xi.U[k], n, Mid, sh.rc, tmp, n, 1.0, 0.0);
        plan_gemm<double>(q, pl, false, true, n, n, sh.rc, tmp, n, lam.U[k], n, dA[j * d + k], n,
                          -op->alpha[j], 0.0);
      }
  }
  fin.add_inputs(sh, op, S, prm->s, omega, sh.sc(), prm);
  fin.alloc(ar);
  finish_blob(ar, blob, st);
  if (ar.measuring()) return 0;
  imp.run(st);
  fin.run(st);
  pre.run(st);
  TT<double> lam;
  SolveInfo si;
  solver_run(*solver, lam, si, st);
  grad[solver_slot_index(*solver)].run(st);
  if (dalpha) {
    TK_HIP(hipMemcpyAsync(dalpha, dal, sizeof(double) * op->nterms, hipMemcpyDeviceToHost, st));
  }
  TK_HIP(hipStreamSynchronize(st));
  if (lambda) export_tt<double>(sh, lam, lambda, hdr, nullptr, nullptr, st);
  fill_info(si, info, d);
  return si.status;
}

// ---------------------------------------------------------------- multilinear Nystrom
void check_mln_rank(int r, int p) {
  TK_CHECK(r >= 1 && r <= 64, kErrUnsupported, "MLN target rank r must be in [1, 64]");
  TK_CHECK(p >= 0 && r + p <= 256, kErrUnsupported, "MLN: need p >= 0 and r + p <= 256");
}

std::array<const double*, kMaxD> psi_of(const double* const* Psi, int d) {
  TK_CHECK(Psi != nullptr, kErrInvalidArg, "Psi is NULL");
  std::array<const double*, kMaxD> a{};
  for (int k = 0; k < d; ++k) a[k] = Psi[k];
  return a;
}

int do_mln_sketch(const tk_block_sum* x, const double* const* Psi, int r, int p, double* core, double* const* F,
                  double* diag, Arena& ar, hipStream_t st) {
  check_mln_rank(r, p);
  Blob blob;
  Planner pl(ar, blob);
  Seq q;
  std::vector<MoveTask<double, double>> mv;
  TK_CHECK(F != nullptr, kErrInvalidArg, "factor sketch outputs missing");
  const Shape shape = shape_of_blocks(x, 1, 0);
  Writes writes = {{core, size_t(ipow(r + p, shape.d))}, {diag, size_t(r + p)}};
  for (int k = 0; k < shape.d; ++k) writes.push_back({F[k], size_t(shape.n[k]) * r});
  const auto im = import_blocks<double>(ar, x, shape, mv, writes);
  emit_moves(q, pl, mv);
  const int d = im.sh.d;
  const auto ps = psi_of(Psi, d);
  MlnSk out;
  out.core = core;
  for (int k = 0; k < d; ++k) out.F[k] = F[k];
  plan_mln_sketch(q, pl, im.sh, im.blocks, ps, r, r + p, out, diag);
  finish_blob(ar, blob, st);
  if (ar.measuring()) return 0;
  TK_CHECK(core != nullptr, kErrInvalidArg, "core output is NULL");
  for (int k = 0; k < d; ++k) {
    TK_CHECK(ps[k] != nullptr, kErrInvalidArg, "Psi factor is NULL");
    TK_CHECK(F[k] != nullptr, kErrInvalidArg, "factor sketch output is NULL");
  }
  q.run(st);
  TK_HIP(hipStreamSynchronize(st));
  return 0;
}

int do_mln_recover(const double* core, const double* const* F, const double* const* Psi, int r, int p, int d,
                   const int64_t* n, tk_tucker* out, Arena& ar, hipStream_t st) {
  check_mln_rank(r, p);
  check_dims(d, n);
  TK_CHECK(F != nullptr, kErrInvalidArg, "factor sketches missing");
  const auto ps = psi_of(Psi, d);
  Shape sh = shape_of(d, n, r, r, p);
  Blob blob;
  Planner pl(ar, blob);
  Seq q;
  MlnSk sk;
  sk.core = const_cast<double*>(core);
  for (int k = 0; k < d; ++k) sk.F[k] = const_cast<double*>(F[k]);
  TT<double> o = alloc_tt<double>(ar, sh);
  int* hdr = ar.alloc<int>(kExportHdr);
  plan_mln_recovery(q, pl, sh, sk, ps, r, r + p, o);
  finish_blob(ar, blob, st);
  if (ar.measuring()) return 0;
  TK_CHECK(core != nullptr && out != nullptr, kErrInvalidArg, "core or output is NULL");
  for (int k = 0; k < d; ++k) {
    TK_CHECK(ps[k] != nullptr && F[k] != nullptr, kErrInvalidArg, "Psi factor or factor sketch is NULL");
    TK_CHECK(out->rcap[k] >= r, kErrCapacity, "output rank capacity below r");
  }
  q.run(st);
  export_tt<double>(sh, o, out, hdr, nullptr, nullptr, st);
  return 0;
}

void check_mln_params(const tk_mln_params* prm) {
  TK_CHECK(prm != nullptr, kErrInvalidArg, "parameters are NULL");
  check_mln_rank(prm->r, prm->p);
  TK_CHECK(prm->tol > 0 && prm->eta > 0 && prm->eta <= 1, kErrInvalidArg, "tol > 0 and 0 < eta <= 1 required");
  TK_CHECK(prm->maxiter >= 1 && prm->maxiter <= 64, kErrUnsupported, "maxiter must be in [1, 64]");
  TK_CHECK(prm->k_trunc >= 1, kErrInvalidArg, "k_trunc must be >= 1");
  TK_CHECK(prm->tikhonov == 0 || prm->tikhonov == 1, kErrInvalidArg, "tikhonov must be 0 or 1");
  if (prm->save_memory)
    TK_CHECK(prm->r_sol >= 1 && prm->r_sol <= prm->r && prm->p_sol >= 0 && prm->r_sol + prm->p_sol <= prm->r + prm->p,
             kErrInvalidArg, "save_memory needs 1 <= r_sol <= r and r_sol + p_sol <= r + p");
  TK_CHECK(prm->precond_q >= 0 && prm->precond_q <= 400, kErrInvalidArg, "precond_q must be in [0, 400]");
  TK_CHECK(prm->precond_q == 0 || (prm->precond_V != nullptr && prm->precond_lambda != nullptr), kErrInvalidArg,
           "preconditioner eigenpairs missing");
}

int do_mln_solve(const tk_kron_op* op, const tk_tucker* b, const tk_mln_params* prm, const double* const* Psi,
                 tk_tucker* x, tk_sgmres_info* info, Arena& ar, hipStream_t st) {
  TK_CHECK(b != nullptr, kErrInvalidArg, "b is NULL");
  check_dims(b->d, b->n);
  check_op(op, b->d, b->n);
  check_tucker(b, "b", b->d, b->n);
  check_mln_params(prm);
  const int d = b->d;
  for (int k = 0; k < d; ++k) TK_CHECK(b->r[k] <= prm->r, kErrCapacity, "rank of b above the target rank r");
  const auto ps = psi_of(Psi, d);
  Shape sh = shape_of(d, b->n, prm->r, prm->r, prm->p);
  Seq imp;
  TT<double> bi = alloc_tt<double>(ar, sh);
  emit_import(imp, sh, *b, bi);
  MlnCfg cfg;
  cfg.r = prm->r;
  cfg.p = prm->p;
  cfg.tol = prm->tol;
  cfg.eta = prm->eta;
  cfg.maxiter = prm->maxiter;
  cfg.k_trunc = prm->k_trunc;
  cfg.bd_tol = prm->breakdown_tol > 0 ? prm->breakdown_tol : 1e-14;
  cfg.save_memory = prm->save_memory != 0;
  cfg.r_sol = prm->r_sol;
  cfg.p_sol = prm->p_sol;
  cfg.tikhonov = prm->tikhonov != 0;
  PrecondT<double> pc;
  pc.q = prm->precond_q;
  if (pc.q > 0)
    for (int k = 0; k < d; ++k) {
      pc.V[k] = prm->precond_V[k];
      pc.lam[k] = prm->precond_lambda[k];
      TK_CHECK(ar.measuring() || (pc.V[k] != nullptr && pc.lam[k] != nullptr), kErrInvalidArg,
               "preconditioner eigenpairs missing");
    }
  int* hdr = ar.alloc<int>(kExportHdr);
  auto solver = make_mln_solver(ar, sh, op_dev(op), bi, cfg, ps, st, pc);
  if (ar.measuring()) return 0;
  TK_CHECK(x != nullptr, kErrInvalidArg, "x is NULL");
  for (int k = 0; k < d; ++k) TK_CHECK(ps[k] != nullptr, kErrInvalidArg, "Psi factor is NULL");
  imp.run(st);
  TT<double> xo;
  MlnInfo mi;
  mln_solver_run(*solver, xo, mi, st);
  export_tt<double>(sh, xo, x, hdr, nullptr, nullptr, st);
  if (info) {
    SolveInfo si;
    si.status = mi.status;
    si.iters = mi.iters;
    si.cycles = 1;
    si.true_relres = mi.true_relres;
    si.seconds = mi.seconds;
    si.hist_sketched = mi.hist;
    si.hist_ranks = mi.ranks;
    si.hist_true = {mi.true_relres};
    si.hist_time = {mi.seconds};
    si.hist_lambda = mi.lambda;
    fill_info(si, info, d);
  }
  return mi.status;
}

// ---------------------------------------------------------------- Tikhonov
int do_tikhonov(const double* M, const double* b, int s, int k, double lam_fixed, double* y, double* out, Arena& ar,
                hipStream_t st) {
  TK_CHECK(k >= 1 && k <= 64, kErrUnsupported, "k must be in [1, 64]");
  TK_CHECK(s >= k && s <= 256, kErrUnsupported, "s must be in [k, 256]");
  TK_CHECK(std::isfinite(lam_fixed) || lam_fixed < 0, kErrInvalidArg, "lambda_fixed must be finite");
  LsState ls{};
  ls.Mcol = M;
  ls.bs = b;
  ls.Hv = ar.alloc<double>(size_t(s) * k);
  ls.tau = ar.alloc<double>(k);
  ls.R = ar.alloc<double>(size_t(k) * k);
  ls.qtb = ar.alloc<double>(s);
  ls.y = ar.alloc<double>(k);
  ls.res = ar.alloc<double>(k);
  ls.nrmM2 = ar.alloc<double>(1);
  ls.flags = ar.alloc<int>(4);
  ls.lam = ar.alloc<double>(k);
  double* bn2 = ar.alloc<double>(1);
  double* bn = ar.alloc<double>(1);
  ls.bs_norm = bn;
  const double** tab = ar.alloc<const double*>(1);
  if (ar.measuring()) return 0;
  TK_CHECK(M != nullptr && b != nullptr && y != nullptr && out != nullptr, kErrInvalidArg, "NULL argument");
  TK_HIP(hipMemcpyAsync(tab, &b, sizeof(b), hipMemcpyHostToDevice, st));
  dot_batched<double>(tab, tab, size_t(s), 1, 1.0, bn2, nullptr, st);
  vec_sqrt(bn2, bn, 1, st);
  ls_init(ls, s, st);
  for (int j = 0; j < k; ++j) ls_add_column(ls, s, k, j, 0.0, 0.0, st);
  ls_tikhonov(ls, s, k, k - 1, 0.0, lam_fixed, st);
  TK_HIP(hipMemcpyAsync(y, ls.y, sizeof(double) * k, hipMemcpyDeviceToDevice, st));
  TK_HIP(hipMemcpyAsync(out, ls.lam + (k - 1), sizeof(double), hipMemcpyDeviceToDevice, st));
  TK_HIP(hipMemcpyAsync(out + 1, ls.res + (k - 1), sizeof(double), hipMemcpyDeviceToDevice, st));
  TK_HIP(hipStreamSynchronize(st));
  return 0;
}

}  // namespace
}  // namespace tk

// ====================================================================== extern "C"
using namespace tk;

static hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

// Static device scratch of the allocation-free sketch entry point.  Each GPU
// the library runs on holds its own copy of this array until the process
// ends.  In host code the array's name is only a host-side stand-in: kernels
// and copies get the device address that hipGetSymbolAddress returns for the
// current device, looked up once per device and kept.
namespace tk {
namespace {
constexpr size_t kNoAllocScratchBytes = size_t(64) << 20;
__device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

void* noalloc_scratch() {
  int dev = -1;
  TK_HIP(hipGetDevice(&dev));
  TK_CHECK(dev >= 0 && dev < kMaxDevices, kErrUnsupported, "device index outside the scratch table");
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    TK_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    TK_CHECK(p != nullptr, kErrHip, "hipGetSymbolAddress returned no address for the static scratch");
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}
}  // namespace
}  // namespace tk

extern "C" {

int tucker_apply_op(const tk_kron_op* op, const tk_tucker* x, int32_t transpose, int32_t form, double* const* AU,
                    void* ws, size_t ws_bytes, void* stream) {
  return guarded([&] {
    TK_CHECK(ws != nullptr || ws_bytes == 0, kErrInvalidArg, "workspace pointer is NULL");
    Arena ar(ws ? ws : reinterpret_cast<void*>(uintptr_t(1)), ws_bytes);
    return do_apply(op, x, transpose, form, AU, ar, as_stream(stream));
  });
}
int tucker_apply_op_workspace(const tk_kron_op* op, const tk_tucker* x, int32_t form, size_t* bytes) {
  return guarded([&] {
    Arena ar(nullptr, 0);
    // one stand-in output per product (the sizes are checked by the plan)
    const size_t np = op && op->nterms > 0 && op->d > 0 ? size_t(op->nterms) * size_t(op->d) : 0;
    std::vector<double*> dummy(np, reinterpret_cast<double*>(uintptr_t(0x1000)));
    const int r = do_apply(op, x, 0, form, dummy.data(), ar, nullptr);
    if (bytes) *bytes = ar.used();
    return r;
  });
}

int tucker_sketch(const tk_block_sum* x, const double* const* S, int64_t s, int32_t form, double* out, void* ws,
                  size_t ws_bytes, void* stream) {
  return guarded([&] {
    TK_CHECK(ws != nullptr, kErrInvalidArg, "workspace pointer is NULL");
    Arena ar(ws, ws_bytes);
    return do_sketch(x, S, s, form, out, ar, as_stream(stream));
  });
}
int tucker_sketch_noalloc(const tk_block_sum* x, const double* const* S, int64_t s, int32_t form, double* out,
                          void* stream) {
  return guarded([&] {
    bool lean = false;
    {
      // size check first, so that an oversized call launches nothing; a plan
      // that is too large is tried again without the buffers of split products
      Arena probe(nullptr, 0);
      do_sketch(x, S, s, form, out, probe, nullptr);
      size_t need = probe.used();
      lean = need > kNoAllocScratchBytes;
      if (lean) {
        Arena small(nullptr, 0);
        do_sketch(x, S, s, form, out, small, nullptr, true);
        need = small.used();
      }
      TK_CHECK(need <= kNoAllocScratchBytes, kErrWorkspace,
               "tucker_sketch_noalloc: needs " + std::to_string(need) +
                   " bytes of scratch, above its static maximum of " + std::to_string(kNoAllocScratchBytes));
    }
    Arena ar(noalloc_scratch(), kNoAllocScratchBytes);
    return do_sketch(x, S, s, form, out, ar, as_stream(stream), lean);
  });
}
int tucker_sketch_workspace(const tk_block_sum* x, int64_t s, int32_t form, size_t* bytes) {
  return guarded([&] {
    Arena ar(nullptr, 0);
    const double* S[TK_MAX_D] = {reinterpret_cast<const double*>(uintptr_t(0x1000)),
                                 reinterpret_cast<const double*>(uintptr_t(0x1000)),
                                 reinterpret_cast<const double*>(uintptr_t(0x1000)),
                                 reinterpret_cast<const double*>(uintptr_t(0x1000))};
    const int r = do_sketch(x, S, s, form, reinterpret_cast<double*>(uintptr_t(0x1000)), ar, nullptr);
    if (bytes) *bytes = ar.used();
    return r;
  });
}

int tucker_rhosvd(const tk_block_sum* in, const tk_round_params* prm, const double* const* omega, tk_tucker* out,
                  int32_t* s_out, void* ws, size_t ws_bytes, void* stream) {
  return guarded([&] {
    TK_CHECK(ws != nullptr, kErrInvalidArg, "workspace pointer is NULL");
    Arena ar(ws, ws_bytes);
    return do_rhosvd(in, prm, omega, out, s_out, ar, as_stream(stream));
  });
}
int tucker_rhosvd_workspace(const tk_block_sum* in, const tk_round_params* prm, size_t* bytes) {
  return guarded([&] {
    Arena ar(nullptr, 0);
    const double* om[TK_MAX_D] = {nullptr, nullptr, nullptr, nullptr};
    const int r = do_rhosvd(in, prm, om, nullptr, nullptr, ar, nullptr);
    if (bytes) *bytes = ar.used();
    return r;
  });
}

int tsgmres_solve(const tk_kron_op* op, const tk_tucker* b, const tk_sgmres_params* prm, const double* const* S,
                  const double* const* omega, tk_tucker* x, tk_sgmres_info* info, void* ws, size_t ws_bytes,
                  void* stream) {
  return guarded([&] {
    TK_CHECK(ws != nullptr, kErrInvalidArg, "workspace pointer is NULL");
    Arena ar(ws, ws_bytes);
    return do_solve(op, b, prm, S, omega, x, info, ar, as_stream(stream));
  });
}
int tsgmres_solve_workspace(const tk_kron_op* op, const tk_tucker* b, const tk_sgmres_params* prm, size_t* bytes) {
  return guarded([&] {
    Arena ar(nullptr, 0);
    const double* dummy[TK_MAX_D] = {nullptr, nullptr, nullptr, nullptr};
    const int r = do_solve(op, b, prm, dummy, dummy, nullptr, nullptr, ar, nullptr);
    if (bytes) *bytes = ar.used();
    return r;
  });
}

int tsgmres_backward(const tk_kron_op* op, const tk_tucker* x, const tk_block_sum* xbar,
                     const tk_sgmres_params* prm, const double* const* S, const double* const* omega,
                     tk_tucker* lambda, double* dalpha, double* const* dA, tk_sgmres_info* info, void* ws,
                     size_t ws_bytes, void* stream) {
  return guarded([&] {
    TK_CHECK(ws != nullptr, kErrInvalidArg, "workspace pointer is NULL");
    Arena ar(ws, ws_bytes);
    return do_backward(op, x, xbar, prm, S, omega, lambda, dalpha, dA, info, ar, as_stream(stream));
  });
}
int tsgmres_backward_workspace(const tk_kron_op* op, const tk_tucker* x, const tk_block_sum* xbar,
                               const tk_sgmres_params* prm, size_t* bytes) {
  return guarded([&] {
    Arena ar(nullptr, 0);
    const double* dummy[TK_MAX_D] = {nullptr, nullptr, nullptr, nullptr};
    std::vector<double*> dA(size_t(op ? op->nterms * op->d : 0), reinterpret_cast<double*>(uintptr_t(0x1000)));
    const int r = do_backward(op, x, xbar, prm, dummy, dummy, nullptr, nullptr, dA.data(), nullptr, ar, nullptr);
    if (bytes) *bytes = ar.used();
    return r;
  });
}

int tucker_norm(const tk_block_sum* x, double* out, void* ws, size_t ws_bytes, void* stream) {
  return guarded([&] {
    TK_CHECK(ws != nullptr, kErrInvalidArg, "workspace pointer is NULL");
    Arena ar(ws, ws_bytes);
    return do_norm(x, out, ar, as_stream(stream));
  });
}
int tucker_norm_workspace(const tk_block_sum* x, size_t* bytes) {
  return guarded([&] {
    Arena ar(nullptr, 0);
    const int r = do_norm(x, nullptr, ar, nullptr);
    if (bytes) *bytes = ar.used();
    return r;
  });
}

int tucker_mln_sketch(const tk_block_sum* x, const double* const* Psi, int32_t r, int32_t p, double* core,
                      double* const* F, double* diag, void* ws, size_t ws_bytes, void* stream) {
  return guarded([&] {
    TK_CHECK(ws != nullptr, kErrInvalidArg, "workspace pointer is NULL");
    Arena ar(ws, ws_bytes);
    return do_mln_sketch(x, Psi, r, p, core, F, diag, ar, as_stream(stream));
  });
}
int tucker_mln_sketch_workspace(const tk_block_sum* x, int32_t r, int32_t p, size_t* bytes) {
  return guarded([&] {
    Arena ar(nullptr, 0);
    // stand-in output addresses: planning only records them (a null core
    // would select a different contraction form)
    double* fake = reinterpret_cast<double*>(uintptr_t(0x1000));
    const double* dummy[TK_MAX_D] = {fake, fake, fake, fake};
    double* F[TK_MAX_D] = {fake, fake, fake, fake};
    const int rv = do_mln_sketch(x, dummy, r, p, fake, F, nullptr, ar, nullptr);
    if (bytes) *bytes = ar.used();
    return rv;
  });
}

int tucker_mln_recover(const double* core, const double* const* F, const double* const* Psi, int32_t r, int32_t p,
                       tk_tucker* out, void* ws, size_t ws_bytes, void* stream) {
  return guarded([&] {
    TK_CHECK(ws != nullptr, kErrInvalidArg, "workspace pointer is NULL");
    TK_CHECK(out != nullptr, kErrInvalidArg, "output is NULL");
    Arena ar(ws, ws_bytes);
    return do_mln_recover(core, F, Psi, r, p, out->d, out->n, out, ar, as_stream(stream));
  });
}
int tucker_mln_recover_workspace(int32_t d, const int64_t* n, int32_t r, int32_t p, size_t* bytes) {
  return guarded([&] {
    TK_CHECK(n != nullptr, kErrInvalidArg, "mode sizes are NULL");
    Arena ar(nullptr, 0);
    const double* dummy[TK_MAX_D] = {nullptr, nullptr, nullptr, nullptr};
    const int rv = do_mln_recover(nullptr, dummy, dummy, r, p, d, n, nullptr, ar, nullptr);
    if (bytes) *bytes = ar.used();
    return rv;
  });
}

int tsgmres_mln_solve(const tk_kron_op* op, const tk_tucker* b, const tk_mln_params* prm, const double* const* Psi,
                      tk_tucker* x, tk_sgmres_info* info, void* ws, size_t ws_bytes, void* stream) {
  return guarded([&] {
    TK_CHECK(ws != nullptr, kErrInvalidArg, "workspace pointer is NULL");
    Arena ar(ws, ws_bytes);
    return do_mln_solve(op, b, prm, Psi, x, info, ar, as_stream(stream));
  });
}
int tsgmres_mln_solve_workspace(const tk_kron_op* op, const tk_tucker* b, const tk_mln_params* prm, size_t* bytes) {
  return guarded([&] {
    Arena ar(nullptr, 0);
    const double* dummy[TK_MAX_D] = {nullptr, nullptr, nullptr, nullptr};
    const int rv = do_mln_solve(op, b, prm, dummy, nullptr, nullptr, ar, nullptr);
    if (bytes) *bytes = ar.used();
    return rv;
  });
}

int tsgmres_projected_tikhonov(const double* M, const double* b, int32_t s, int32_t k, double lambda_fixed,
                               double* y, double* out, void* ws, size_t ws_bytes, void* stream) {
  return guarded([&] {
    TK_CHECK(ws != nullptr, kErrInvalidArg, "workspace pointer is NULL");
    Arena ar(ws, ws_bytes);
    return do_tikhonov(M, b, s, k, lambda_fixed, y, out, ar, as_stream(stream));
  });
}
int tsgmres_projected_tikhonov_workspace(int32_t s, int32_t k, size_t* bytes) {
  return guarded([&] {
    Arena ar(nullptr, 0);
    const int rv = do_tikhonov(nullptr, nullptr, s, k, -1.0, nullptr, nullptr, ar, nullptr);
    if (bytes) *bytes = ar.used();
    return rv;
  });
}

int tk_kernel_timer(int32_t kind, int32_t enable) {
  return guarded([&] {
    TK_CHECK(kind >= 0 && kind < kKcCount, kErrInvalidArg, "unknown kernel class");
    timer_enable(kind, enable != 0);
    return 0;
  });
}
int tk_kernel_timer_read(int32_t kind, int64_t* launches, double* total_ms, double* flops, double* bytes) {
  return guarded([&] {
    TK_CHECK(kind >= 0 && kind < kKcCount && launches && total_ms, kErrInvalidArg, "bad timer query");
    double f = 0.0, b = 0.0;
    timer_read(kind, launches, total_ms, &f, &b);
    if (flops) *flops = f;
    if (bytes) *bytes = b;
    return 0;
  });
}

int tk_launch_count(int64_t* count) {
  return guarded([&] {
    TK_CHECK(count != nullptr, kErrInvalidArg, "count is NULL");
    *count = launch_count();
    return 0;
  });
}
int tk_launch_latency(int32_t n, void* stream, double* us_per_launch) {
  return guarded([&] {
    TK_CHECK(n >= 1 && n <= 1000000 && us_per_launch != nullptr, kErrInvalidArg, "bad launch-latency query");
    *us_per_launch = empty_launch_us(n, as_stream(stream));
    return 0;
  });
}

int tk_rank_cert_count(int64_t* tried, int64_t* passed) {
  return guarded([&] {
    TK_CHECK(tried != nullptr && passed != nullptr, kErrInvalidArg, "count pointer is NULL");
    rank_cert_counts(tried, passed);
    return 0;
  });
}

const char* tk_last_error(void) { return tk::last_error(); }
int tk_version(void) { return TK_ABI_VERSION; }

}  // extern "C"
