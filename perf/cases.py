"""Performance cases of the Tucker sGMRES framework: the calls that a program
built on it makes, from the smallest per-step call to whole solves, with their
inputs drawn on the GPU from a seed.

Interface: ``listed()`` (the fixed cases), ``draw(rng)`` (one more case of the
same ranges), ``prepare(case, seed)`` (what the program holds before the
call), ``run(state)`` (one pass through the public entry points),
``work(case)`` (bytes and flops the path cannot do without) and
``exact(case, seed)`` (the pass's outputs in plain float64 NumPy where they
have such a value).

Operators are those of the workload generators: the 3D Poisson operator, 3D
convection-diffusion (six Kronecker terms), the deblurring operator
``M x M x M + 1e-3 I`` and the 4D Poisson operator with two Kronecker
perturbations.  Basis-like Tucker tensors have orthonormal factors and cores
whose singular values decay geometrically, as the solver's basis tensors do.

A Tucker tensor is only determined up to the signs and rotations of its
factors, so a case whose result is one reads it out on fixed measurement
functions (``project_core``: the tensor contracted with m functions a mode),
which determines it when m is at least its ranks; ranks and sketch widths come
back as whole numbers.  The FP32 and BF16-factor forms return float64 buffers
with FP32 content; their results are kept as float32, as a program of that
form would.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2608_11091_amd as tk
from workloads import (centered_difference_1d, gaussian_blur_toeplitz, laplacian_1d, laplacian_eigenpairs)


def listed():
    return [
        # one operator application of the smallest workload (Poisson n = 32,
        # rank 10): launch and host latency of a per-step call
        dict(name="apply_poisson_n32", kind="apply", op="poisson", n=32, ragged=False, r=10, transpose=False, form=0),
        # transposed application of the six-term convection-diffusion operator
        # at its configured size, as in every adjoint iteration
        dict(name="apply_convdiff_n256_t", kind="apply", op="convdiff", n=256, ragged=False, r=32, transpose=True,
             form=0),
        # Khatri-Rao sketch (s = 120) of L(X), six blocks, convection-diffusion
        dict(name="sketch_convdiff_n256", kind="sketch", op="convdiff", n=256, ragged=False, r=32, s=120, form=0),
        # orthogonalisation RoundSum of three small tensors (Poisson n = 32, cap 10)
        dict(name="round_poisson_n32", kind="round", op="", d=3, n=32, ragged=False, blocks=3, r=10, cap=10, p=5,
             form=0),
        # the same at odd, unequal mode sizes: rank below the cap, both prime
        dict(name="round_ragged_n173", kind="round", op="", d=3, n=173, ragged=True, blocks=2, r=23, cap=31, p=6,
             form=0),
        # orthogonalisation RoundSum of the deblurring benchmark (three
        # rank-48 blocks, n = 512), FP64 form
        dict(name="round_deblur_n512", kind="round", op="", d=3, n=512, ragged=False, blocks=3, r=48, cap=48, p=5,
             form=0),
        # RoundSum of L(V) of the same workload in the FP32 form, the form of
        # the benchmark's cycles
        dict(name="round_deblur_n512_f32", kind="round", op="deblur", d=3, n=512, ragged=False, blocks=2, r=48,
             cap=48, p=5, form=1),
        # RoundSum of L(V) of the four-dimensional workload (six blocks of rank 32)
        dict(name="round_poisson4d_n128", kind="round", op="poisson4d", d=4, n=128, ragged=False, blocks=6, r=32,
             cap=32, p=5, form=0),
        # multilinear Nystrom sketch and recovery at the benchmark's size (r = p = 48)
        dict(name="mln_deblur_n512", kind="mln", op="deblur", n=512, ragged=False, r=48, p=48),
        # the first twelve iterations of the deblurring benchmark's cycle with
        # the final assembly and the true residual, FP64 form
        dict(name="solve_deblur_n512", kind="solve", op="deblur", n=512, cap=48, p=5, s=120, maxiter=12, method=0),
        # MLN-Tucker sGMRES on convection-diffusion, twenty iterations
        dict(name="mln_solve_convdiff_n256", kind="mln_solve", op="convdiff", n=256, r=32, p=32, maxiter=20),
        # a training step: preconditioned forward solve, loss, adjoint solve
        # and gradients with respect to alpha and the core of b
        dict(name="loss_poisson_n128", kind="loss", op="poisson", n=128, cap=32, p=5, q=36),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["apply", "sketch", "round", "round", "round", "mln", "solve", "mln_solve", "loss"])
    op = rng.choice(["poisson", "convdiff", "deblur"])
    if kind == "apply":
        n = _log(rng, 16, 512)
        return dict(kind=kind, op=op, n=n, ragged=rng.random() < 0.5, r=min(n - 8, _log(rng, 2, 64)),
                    transpose=rng.random() < 0.5, form=rng.choice([0, 0, 1, 2]))
    if kind == "sketch":
        n = _log(rng, 16, 512)
        return dict(kind=kind, op=op, n=n, ragged=rng.random() < 0.5, r=min(n - 8, _log(rng, 2, 48)),
                    s=_log(rng, 20, 256), form=rng.choice([0, 0, 1, 2]))
    if kind == "round":
        d = 4 if rng.random() < 0.2 else 3
        n = _log(rng, 16, 128 if d == 4 else 512)
        p = rng.randint(3, 8)
        cap = min(n - 8, _log(rng, 5, 32 if d == 4 else 48))
        return dict(kind=kind, op=rng.choice(["", "", "convdiff", "deblur"]) if d == 3 else "", d=d, n=n,
                    ragged=rng.random() < 0.5, blocks=rng.randint(1, 4), r=max(2, int(cap * rng.uniform(0.5, 1.0))),
                    cap=cap, p=min(p, n - 8 - cap) if n - 8 - cap > 0 else 1, form=rng.choice([0, 0, 1]))
    if kind == "mln":
        n = _log(rng, 40, 512)
        r = min(n // 3, _log(rng, 4, 48))
        return dict(kind=kind, op=op, n=n, ragged=rng.random() < 0.5, r=r, p=max(2, int(r * rng.uniform(0.5, 1.0))))
    if kind == "solve":
        n = _log(rng, 24, 512)
        return dict(kind=kind, op=op, n=n, cap=min(n // 2, _log(rng, 8, 40)), p=5, s=rng.randint(40, 160),
                    maxiter=rng.randint(3, 9), method=rng.choice([0, 0, 1]))
    if kind == "mln_solve":
        n = _log(rng, 48, 256)
        r = min(n // 3, _log(rng, 8, 32))
        return dict(kind=kind, op="convdiff", n=n, r=r, p=r, maxiter=rng.randint(3, 12))
    return dict(kind="loss", op="poisson", n=_log(rng, 24, 128), cap=rng.randint(24, 32), p=5, q=36)


# ---------------------------------------------------------------- inputs
def _modes(case):
    d = case.get("d", 3)
    n = case["n"]
    return [n - (0, 3, 7, 2)[k] for k in range(d)] if case.get("ragged") else [n] * d


def _terms(op, ns):
    """Kronecker terms of the workload's operator as NumPy matrices."""
    d = len(ns)
    if op == "poisson":
        return [(1.0, [laplacian_1d(n) if j == k else None for j, n in enumerate(ns)]) for k in range(d)]
    if op == "convdiff":
        t = [(1e-2, [laplacian_1d(n) if j == k else None for j, n in enumerate(ns)]) for k in range(d)]
        return t + [(c, [centered_difference_1d(n) if j == k else None for j, n in enumerate(ns)])
                    for k, c in zip(range(d), (1.0, 0.5, 0.25, 0.125))]
    if op == "deblur":
        M = {n: gaussian_blur_toeplitz(n).T @ gaussian_blur_toeplitz(n) for n in set(ns)}
        return [(1.0, [M[n] for n in ns]), (1e-3, [None] * d)]
    if op == "poisson4d":
        rng = np.random.default_rng(1)
        t = [(1.0, [laplacian_1d(n) if j == k else None for j, n in enumerate(ns)]) for k in range(d)]
        for _ in range(2):
            t.append((1.0, [np.eye(n) + 0.01 / math.sqrt(n) * rng.standard_normal((n, n)) for n in ns]))
        return t
    raise ValueError(op)


def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + salt)
    return g


def _normal(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)


def _tensor(g, ns, r, decay=1e-4):
    """Basis-like Tucker tensor: orthonormal factors, core entries N(0, 1)
    scaled by decay^((i_1 + ... + i_d) / r), unit norm."""
    d = len(ns)
    U = [torch.linalg.qr(_normal(g, n, r))[0].t().contiguous() for n in ns]
    i = torch.arange(r, device="cuda", dtype=torch.float64)
    w = decay ** (i / r)
    core = _normal(g, *([r] * d))
    for k in range(d):
        core = core * w.reshape([-1 if j == k else 1 for j in range(d)])
    return tk.Tucker((core / core.norm()).contiguous(), U, (r,) * d)


def _smooth(g, ns, r, modes):
    """Tucker tensor of rank r whose factors combine the lowest sine modes."""
    U = []
    for n in ns:
        i = torch.arange(1, n + 1, device="cuda", dtype=torch.float64)
        j = torch.arange(1, modes + 1, device="cuda", dtype=torch.float64)
        sines = torch.sin(torch.outer(i, j) * math.pi / (n + 1)) * math.sqrt(2.0 / (n + 1))
        U.append((sines @ (_normal(g, modes, r) / j[:, None])).t().contiguous())
    return tk.Tucker(_normal(g, *([r] * len(ns))), U, (r,) * len(ns))


def _measure_width(case):
    return 16 if case.get("d", 3) == 4 else min(48, min(_modes(case)))


def _sketches(g, ns, s, w):
    return [_normal(g, s, n) for n in ns], [_normal(g, w, n) for n in ns]


def prepare(case, seed):
    kind, ns = case["kind"], _modes(case)
    g = _gen(seed, 17)
    st = dict(case=case)
    if kind not in ("loss",) and case["op"]:
        st["op"] = tk.KronOp.from_terms(_terms(case["op"], ns))
    if kind == "apply":
        st["x"] = _tensor(g, ns, case["r"])
    elif kind == "sketch":
        x = _tensor(g, ns, case["r"])
        st["blocks"] = tk.apply_op(st["op"], x)
        st["S"] = _sketches(g, ns, case["s"], 1)[0]
    elif kind == "round":
        if case["op"]:
            # L(V), as the solver rounds it after every application
            st["blocks"] = tk.apply_op(st["op"], _tensor(g, ns, case["r"]))
        else:
            # W - sum_j h_j V_j of the orthogonalisation
            h = [1.0, -0.7, 0.4, -0.2]
            st["blocks"] = [(h[b], _tensor(g, ns, case["r"])) for b in range(case["blocks"])]
        st["omega"] = [_normal(g, case["cap"] + case["p"], n) for n in ns]
    elif kind == "mln":
        st["blocks"] = tk.apply_op(st["op"], _tensor(g, ns, case["r"]))
        st["Psi"] = [_normal(g, case["r"] + case["p"], n) for n in ns]
    elif kind == "solve":
        st["b"] = _tensor(g, ns, 5)
        st["S"], st["omega"] = _sketches(g, ns, case["s"], case["cap"] + case["p"])
        # one cycle of a fixed number of iterations (the tolerance is out of reach)
        st["prm"] = tk.SolveParams(form=0, tol=1e-12, maxiter=case["maxiter"], max_restarts=1, k_trunc=2,
                                   rank_cap=case["cap"], oversample=case["p"], eps_trunc=1e-12,
                                   method=case["method"])
    elif kind == "mln_solve":
        st["b"] = _tensor(g, ns, 3)
        st["Psi"] = [_normal(g, case["r"] + case["p"], n) for n in ns]
        st["prm"] = tk.MlnParams(r=case["r"], p=case["p"], tol=1e-12, maxiter=case["maxiter"], k_trunc=2)
    elif kind == "loss":
        alpha = [0.8, 1.4, 0.6]
        cap, p = case["cap"], case["p"]
        L = laplacian_1d(case["n"])
        V, lam = laplacian_eigenpairs(ns)
        S, omega = _sketches(g, ns, 80, cap + p)
        st["problem"] = dict(
            op=tk.KronOp.from_terms([(a, [L if j == k else None for j in range(3)]) for k, a in enumerate(alpha)]),
            b=_smooth(g, ns, 4, 6), x_target=_smooth(g, ns, 3, 6), S=S, omega=omega,
            prm=tk.SolveParams(form=0, tol=1e-8, maxiter=40, k_trunc=2, rank_cap=cap, oversample=p, max_restarts=8,
                               eps_trunc=1e-12, precond_q=case["q"],
                               precond=tk.precond_tensors(V, [l * a for l, a in zip(lam, alpha)])))
        st["alpha"] = torch.tensor(alpha, dtype=torch.float64, device="cuda", requires_grad=True)
        st["core"] = st["problem"]["b"].core.clone().requires_grad_(True)
    if kind in ("round", "mln", "solve", "mln_solve"):
        st["phi"] = [_normal(g, _measure_width(case), n) / math.sqrt(n) for n in ns]
    return st


# ---------------------------------------------------------------- one pass
def _kept(x, form):
    return x.float() if form else x


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "apply":
        blocks = tk.apply_op(st["op"], st["x"], transpose=case["transpose"], form=case["form"])
        return [[_kept(u, case["form"]) for u, A in zip(t.U, As) if A is not None]
                for (_, t), As in zip(blocks, st["op"].A)]
    if kind == "sketch":
        return _kept(tk.sketch(st["blocks"], st["S"], form=case["form"]), case["form"])
    if kind == "round":
        w, s = tk.rhosvd(st["blocks"], st["omega"], _eps(case), case["cap"], case["p"], form=case["form"])
        return dict(values=_kept(tk.project_core(w, st["phi"]), case["form"]), ranks=list(w.ranks), width=s)
    if kind == "mln":
        core, F, diag = tk.mln_sketch(st["blocks"], st["Psi"], case["r"])
        w = tk.mln_recover(core, F, st["Psi"], case["r"])
        return dict(core=core, F=F, diag=diag, values=tk.project_core(w, st["phi"]), ranks=list(w.ranks))
    if kind == "solve":
        x, info = tk.solve(st["op"], st["b"], st["S"], st["omega"], st["prm"])
        return dict(values=tk.project_core(x, st["phi"]), hist=np.array(info["hist"]), iters=info["iters"])
    if kind == "mln_solve":
        x, info = tk.mln_solve(st["op"], st["b"], st["Psi"], st["prm"])
        return dict(values=tk.project_core(x, st["phi"]), hist=np.array(info["hist"]), iters=info["iters"])
    st["alpha"].grad = st["core"].grad = None
    loss = tk.TuckerSGMRESLoss.apply(st["alpha"], st["core"], st["problem"])
    loss.backward()
    return dict(loss=loss.detach(), alpha=st["alpha"].grad, core=st["core"].grad)


def _eps(case):
    return 1e-6 if case["form"] else 1e-10


# ---------------------------------------------------------------- least work
def _products(case, ns):
    """(distinct operator factors, blocks of L(x))"""
    d = len(ns)
    return {"poisson": (d, d), "convdiff": (2 * d, 2 * d), "deblur": (d, 2), "poisson4d": (3 * d, d + 2),
            "": (0, case.get("blocks", 1))}[case["op"]]


def _round_flops(ns, T, r, s):
    """Range sketch, its QR, core projection and ST-HOSVD of T rank-r blocks at sketch width s."""
    d = len(ns)
    f = sum(T * 4.0 * n * r * s + 4.0 * n * s * s + T * 2.0 * n * r * s for n in ns)
    f += T * d * 2.0 * r ** d * s + T * sum(2.0 * s ** m * r ** (d - m + 1) for m in range(1, d + 1))
    return f + d * (4.0 * s ** (d + 1) + 9.0 * s ** 3)


def work(case):
    ns = _modes(case)
    d, sn = len(ns), sum(ns)
    nf, T = _products(case, ns)
    z = 4 if case.get("form") else 8
    kind = case["kind"]
    if kind == "apply":
        r = case["r"]
        per = nf / d
        return dict(bytes=8.0 * sum(per * n * n + n * r + per * n * r for n in ns),
                    flops=sum(per * 2.0 * n * n * r for n in ns))
    if kind == "sketch":
        r, s = case["r"], case["s"]
        return dict(bytes=8.0 * (r ** d + sn * s + (1 + nf / d) * sn * r + s),
                    flops=T * (2.0 * sn * r * s + 2.0 * r ** d * s))
    if kind == "round":
        r, s = case["r"], case["cap"] + case["p"]
        cores = 1 if case["op"] else T
        facs = 1 + nf / d if case["op"] else T
        return dict(bytes=8.0 * (cores * r ** d + facs * sn * r + sn * s + case["cap"] ** d + sn * case["cap"]),
                    flops=_round_flops(ns, T, r, min(s, min(ns))))
    if kind == "mln":
        r, rt = case["r"], case["r"] + case["p"]
        f = T * (sn * 2.0 * r * (r + rt) + d * 2.0 * r ** d * r + sum(2.0 * rt ** m * r ** (d - m + 1) for m in
                                                                       range(1, d + 1)))
        f += sn * 2.0 * r * r * 2 + sn * 2.0 * rt * r + d * 8.0 * rt * r * r
        f += sum(2.0 * rt ** m * r ** (d - m + 1) for m in range(1, d + 1))
        return dict(bytes=8.0 * (r ** d + (1 + nf / d) * sn * r + sn * rt + rt ** d + sn * r + r ** d + sn * r), flops=f)
    if kind == "solve":
        r, s, it = case["cap"], case["cap"] + case["p"], case["maxiter"]
        win = it / 2 if case["method"] else 2
        per = nf / d * sum(2.0 * n * n * r for n in ns) + _round_flops(ns, T, r, s) + _round_flops(ns, 1 + win, r, s)
        per += win * (2.0 * sn * r * r + 2.0 * d * r ** (d + 1))
        if not case["method"]:
            per += 2.0 * sn * r * case["s"] + 2.0 * r ** d * case["s"]
        io = nf / d * sum(n * n for n in ns) + sn * (s + case["s"] + 2 * r) + 2 * r ** d
        basis = it * (sn * r + r ** d)  # every basis tensor written once and read by the final sum
        return dict(bytes=8.0 * (io + 2 * basis), flops=it * per + _round_flops(ns, it, r, s))
    if kind == "mln_solve":
        r, rt, it = case["r"], case["r"] + case["p"], case["maxiter"]
        sketch = sn * 2.0 * r * (r + rt) + d * 2.0 * r ** (d + 1)
        sketch += sum(2.0 * rt ** m * r ** (d - m + 1) for m in range(1, d + 1))
        rec = sn * 2.0 * rt * r + sn * 2.0 * r * r + d * 8.0 * rt * r * r
        rec += sum(2.0 * rt ** m * r ** (d - m + 1) for m in range(1, d + 1))
        per = nf / d * sum(2.0 * n * n * r for n in ns) + (T + 1) * sketch + 2 * rec
        io = nf / d * sum(n * n for n in ns) + sn * (rt + 2 * r) + 2 * r ** d
        return dict(bytes=8.0 * (io + 2 * it * (rt ** d + sn * r)), flops=it * per)
    # loss: forward and adjoint preconditioned solves of about three iterations each
    r, s, terms = case["cap"], case["cap"] + case["p"], 2 * case["q"] + 1
    per = sum(6.0 * n * n * r for n in ns) + _round_flops(ns, terms, r, s) + _round_flops(ns, 3, r, s) * 2
    io = 2 * sum(2 * n * n for n in ns) + 2 * sn * (s + 80) + 4 * (sn * r + r ** d)
    return dict(bytes=8.0 * io, flops=6 * per)


# ---------------------------------------------------------------- 64-bit values
def _np(t):
    return t.detach().double().cpu().numpy()


def _np_tucker(x):
    r = x.ranks
    core = _np(x.core)[tuple(slice(0, v) for v in r)]
    return core, [_np(u)[:v].T for u, v in zip(x.U, r)]


def _ttm(core, mats):
    for k, m in enumerate(mats):
        core = np.moveaxis(np.tensordot(m, core, axes=([1], [k])), 0, k)
    return core


def _unfold(x, k):
    return np.moveaxis(x, k, 0).reshape(x.shape[k], -1)


def _krp(mats):
    out = mats[0]
    for m in mats[1:]:
        out = (out[:, None, :] * m[None, :, :]).reshape(-1, out.shape[1])
    return out


def _range_sketch(blocks, L, k):
    y = 0.0
    for c, core, U in blocks:
        m = [u.T @ l for u, l in zip(U, L)]
        y = y + c * (U[k] @ (_unfold(core, k) @ _krp([m[j] for j in range(len(U)) if j != k])))
    return y


def _np_blocks(blocks):
    return [(c,) + _np_tucker(t) for c, t in blocks]


def _round64(blocks, omega, eps, cap, p):
    """RoundSum in float64: effective-rank width, Khatri-Rao range finder, core, sequentially truncated HOSVD."""
    d = len(omega)
    w = [abs(c) * np.linalg.norm(core) for c, core, _ in blocks]
    rt = 0
    for k in range(d):
        cat = np.concatenate([wb * U[k] for wb, (_, _, U) in zip(w, blocks)], axis=1)
        lam = np.linalg.eigvalsh(cat.T @ cat if cat.shape[1] < cat.shape[0] else cat @ cat.T)[::-1]
        lam = np.where(lam > 1e-12 * lam[0], lam, 0.0)
        tail = np.cumsum(lam[::-1])[::-1]
        rt = max(rt, int(np.sum(tail > eps * eps * lam.sum())))
    s = min(rt + p, cap + p)
    Q = [np.linalg.qr(_range_sketch(blocks, [o[:, :s] for o in omega], k))[0] for k in range(d)]
    core = sum(c * _ttm(G, [q.T @ u for q, u in zip(Q, U)]) for c, G, U in blocks)
    total = np.linalg.norm(core) ** 2
    ranks = []
    for k in range(d):
        u, sv, _ = np.linalg.svd(_unfold(core, k), full_matrices=False)
        tail = np.cumsum(sv[::-1] ** 2)[::-1]
        r = max(1, min(int(np.sum(tail > eps * eps * total / d)), cap))
        core = np.moveaxis(np.tensordot(u[:, :r].T, core, axes=([1], [k])), 0, k)
        Q[k] = Q[k] @ u[:, :r]
        ranks.append(r)
    return core, Q, ranks, s


def exact(case, seed):
    kind = case["kind"]
    if kind in ("solve", "mln_solve"):
        return None  # unconverged Krylov iterates: no closed form
    ns = _modes(case)
    st = prepare(case, seed)
    if kind == "apply":
        _, U = _np_tucker(st["x"])
        out = []
        for _, As in _terms(case["op"], ns):
            out.append([((A.T if case["transpose"] else A) @ u).T for A, u in zip(As, U) if A is not None])
        return out
    if kind == "loss":
        return _loss64(st)
    blocks = _np_blocks(st["blocks"])
    if kind == "sketch":
        S = [_np(t).T for t in st["S"]]
        out = 0.0
        for c, core, U in blocks:
            m = [u.T @ l for u, l in zip(U, S)]
            out = out + c * np.einsum("pl,pl->l", core.reshape(-1, core.shape[-1]) @ m[-1], _krp(m[:-1]))
        return out
    phi = [_np(t).T for t in st["phi"]]
    if kind == "round":
        core, Q, ranks, s = _round64(blocks, [_np(t).T for t in st["omega"]], _eps(case), case["cap"], case["p"])
        return dict(values=_ttm(core, [f.T @ q for f, q in zip(phi, Q)]), ranks=None, width=None)
    Psi = [_np(t).T for t in st["Psi"]]
    r = case["r"]
    core = sum(c * _ttm(G, [P.T @ u for P, u in zip(Psi, U)]) for c, G, U in blocks)
    F = [_range_sketch(blocks, [P[:, :r] for P in Psi], k) for k in range(3)]
    rec = _ttm(core, [f.T @ (Fk @ np.linalg.pinv(P.T @ Fk, rcond=1e-12)) for f, Fk, P in zip(phi, F, Psi)])
    i = np.arange(r + case["p"])
    return dict(core=core, F=[f.T for f in F], diag=core[i, i, i], values=rec, ranks=None)


def _loss64(st):
    """Loss and gradients through the sine transform of the dense tensors."""
    p = st["problem"]
    alpha = _np(st["alpha"])
    bc, bU = _np_tucker(p["b"])
    tc, tU = _np_tucker(p["x_target"])
    V, lam = laplacian_eigenpairs([u.shape[0] for u in bU])
    vb = [v.T @ u for v, u in zip(V, bU)]
    parts = [a * l.reshape([-1 if j == k else 1 for j in range(3)]) for k, (a, l) in enumerate(zip(alpha, lam))]
    den = parts[0] + parts[1] + parts[2]
    x = _ttm(bc, vb) / den
    r = x - _ttm(tc, [v.T @ u for v, u in zip(V, tU)])
    adj = r / den
    da = np.array([-np.sum(adj * x * parts[k]) / alpha[k] for k in range(3)])
    return dict(loss=np.array(0.5 * np.sum(r * r)), alpha=da, core=_ttm(adj, [v.T for v in vb]))
