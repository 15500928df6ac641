"""Moves between caller tensors and internal buffers: one launch brings in the
cores, factors and ranks of every block (capacities above the ranks, unequal
per mode and per block), one exports the result into capacities of its own,
and the factor products of an operator are grouped by shape.  The moves are
copies, so a sketch equals the float64 contraction to rounding (1e-12; 2e-5
for the FP32 form) and the exported padding is exactly zero; an output that is
too small is refused and stays untouched."""
import ctypes as C

import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def tk():
    import paper_2608_11091_amd as tk
    tk.load()
    return tk


def _cm(M):
    return torch.from_numpy(np.ascontiguousarray(M.T)).cuda()


def _blocks(rng, ns, ranks, pads):
    out = []
    for r, pad in zip(ranks, pads):
        core = rng.standard_normal(r)
        U = [np.linalg.qr(rng.standard_normal((n, k)))[0] for n, k in zip(ns, r)]
        out.append((float(rng.uniform(0.5, 1.5)), core, U, tuple(k + q for k, q in zip(r, pad))))
    return out


CASES = [((9, 5), [(1, 1)], [(0, 0)], 3),
         ((40, 33), [(5, 4), (2, 7)], [(0, 3), (9, 1)], 12),
         ((24, 17, 31), [(3, 1, 5)], [(2, 4, 0)], 7),
         ((16, 16, 16), [(4, 4, 4), (2, 5, 3), (1, 5, 5)], [(0, 0, 0), (6, 1, 4), (3, 3, 0)], 14),
         ((8, 13, 11, 9), [(2, 3, 1, 4), (3, 2, 2, 1)], [(1, 0, 3, 0), (0, 2, 1, 4)], 6)]


@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("ns,ranks,pads,cap", CASES)
def test_import_export(tk, ns, ranks, pads, cap, form):
    rng = np.random.default_rng(sum(ns) + len(ranks))
    X = _blocks(rng, ns, ranks, pads)
    blocks = []
    for c, core, U, rcap in X:
        t = tk.Tucker.from_numpy(core, U, rcap=rcap)
        for k, u in enumerate(t.U):  # what lies beyond the ranks is not read
            u[core.shape[k]:] = 7.0
        blocks.append((c, t))
    dense = sum(c * np.einsum("".join("abcd"[k] for k in range(len(ns))) + "," +
                              ",".join("wxyz"[k] + "abcd"[k] for k in range(len(ns))) + "->" + "wxyz"[:len(ns)],
                              core, *U) for c, core, U, _ in X)
    S = [rng.standard_normal((n, 10)) for n in ns]
    ref = np.einsum("wxyz"[:len(ns)] + "," + ",".join("wxyz"[k] + "s" for k in range(len(ns))) + "->s", dense, *S)
    tol = 2e-5 if form else 1e-12
    got = tk.sketch(blocks, [_cm(a) for a in S], form=form).cpu().numpy()
    assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref) * (1 if form == 0 else 2)

    om = [_cm(rng.standard_normal((n, cap + 2))) for n in ns]
    rc = tuple(cap + 3 - k for k in range(len(ns)))
    w, s = tk.rhosvd(blocks, om, 1e-4 if form else 1e-10, cap, 2, out_rcap=rc, form=form)
    assert w.rcap == rc and 1 <= s <= cap + 2
    core, U = w.core.cpu().numpy(), [u.cpu().numpy() for u in w.U]
    inner = core[tuple(slice(0, r) for r in w.ranks)].copy()
    core[tuple(slice(0, r) for r in w.ranks)] = 0.0
    assert not core.any() and all(not u[r:].any() for u, r in zip(U, w.ranks))
    got = inner
    for k, (u, r) in enumerate(zip(U, w.ranks)):
        got = np.moveaxis(np.tensordot(u[:r].T, got, axes=([1], [k])), 0, k)
    err = np.linalg.norm(got - dense) / np.linalg.norm(dense)
    print(f"import/export {ns} form {form}: ranks {w.ranks} err {err:.1e}", flush=True)
    assert err <= (2e-4 if form else 2e-10)


def test_small_output_is_refused_untouched(tk):
    from paper_2608_11091_amd import _abi
    rng = np.random.default_rng(3)
    (c, core, U, rcap), = _blocks(rng, (20, 20, 20), [(6, 6, 6)], [(0, 0, 0)])
    X = [(c, tk.Tucker.from_numpy(core, U))]
    om = [_cm(rng.standard_normal((20, 10))) for _ in range(3)]
    lib = _abi.load()
    from paper_2608_11091_amd import api
    bs, keep = api._blocks_struct(X)
    prm = api.TkRoundParams()
    prm.eps, prm.tau, prm.rank_cap, prm.oversample, prm.force_s, prm.form = 1e-10, -1.0, 8, 2, -1, 0
    for k in range(api.TK_MAX_D):
        prm.force_ranks[k] = -1
    out = tk.Tucker.empty((20, 20, 20), (8, 3, 8))
    out.core += 5.0
    for u in out.U:
        u += 5.0
    os_ = out.struct()
    nb = C.c_size_t()
    assert lib.tucker_rhosvd_workspace(C.byref(bs), C.byref(prm), C.byref(nb)) == 0
    ws = api._workspace(nb.value, out.core.device)
    s = C.c_int32(0)
    rc = lib.tucker_rhosvd(C.byref(bs), C.byref(prm), api._ptr_array(om), C.byref(os_), C.byref(s),
                           C.c_void_p(ws.data_ptr()), nb.value, api._stream())
    torch.cuda.synchronize()
    assert rc != 0
    assert bool((out.core == 5.0).all()) and all(bool((u == 5.0).all()) for u in out.U)


@pytest.mark.parametrize("transpose", [False, True])
@pytest.mark.parametrize("form,tol", [(0, 1e-13), (1, 1e-5), (2, 2e-2)])
@pytest.mark.parametrize("ns,r,rcap", [((7,) * 3, (2, 3, 4), (5, 5, 5)), ((33, 20, 33), (6, 6, 2), (6, 7, 6)),
                                       ((64, 65, 64, 12), (3, 3, 3, 3), (3, 3, 4, 3))])
def test_grouped_products(tk, ns, r, rcap, form, tol, transpose):
    rng = np.random.default_rng(sum(ns))
    x = tk.Tucker.from_numpy(rng.standard_normal(r), [rng.standard_normal((n, k)) for n, k in zip(ns, r)], rcap=rcap)
    shared = {n: rng.standard_normal((n, n)) for n in set(ns)}
    terms = [(1.0 + j, [shared[n] if j == k else (rng.standard_normal((n, n)) if j == len(ns) else None)
                        for k, n in enumerate(ns)]) for j in range(len(ns) + 1)]
    blocks = tk.apply_op(tk.KronOp.from_terms(terms), x, transpose=transpose, form=form)
    for (c, As), (a, y) in zip(terms, blocks):
        assert a == c
        for k, A in enumerate(As):
            u = x.U[k].cpu().numpy()
            ref = u if A is None else u @ (A if transpose else A.T)
            got = y.U[k].cpu().numpy()
            assert got.shape == ref.shape
            if A is not None:
                assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)


def test_sketch_into_its_inputs(tk):
    """Outputs that lie in the inputs' own storage: the inputs are then copied
    before anything is written, so the result is that of separate outputs."""
    import ctypes as C

    from paper_2608_11091_amd import _abi, api
    rng = np.random.default_rng(9)
    n, r, p = 24, 6, 2
    x = tk.Tucker.from_numpy(rng.standard_normal((r,) * 3), [rng.standard_normal((n, r)) for _ in range(3)])
    Psi = [_cm(rng.standard_normal((n, r + p))) for _ in range(3)]
    core, F, diag = tk.mln_sketch([(1.5, x)], Psi, r)
    bs, keep = api._blocks_struct([(1.5, x)])
    lib = _abi.load()
    out = torch.zeros_like(core)
    nb = C.c_size_t()
    api.check(lib.tucker_mln_sketch_workspace(C.byref(bs), r, p, C.byref(nb)))
    ws = api._workspace(nb.value, core.device)
    api.check(lib.tucker_mln_sketch(C.byref(bs), api._ptr_array(Psi), r, p, C.c_void_p(out.data_ptr()),
                                    api._ptr_array(x.U), None, C.c_void_p(ws.data_ptr()), nb.value, api._stream()))
    assert torch.equal(out, core) and all(torch.equal(u, f) for u, f in zip(x.U, F))


def test_workspace_does_not_depend_on_ranks(tk):
    """Blocks with and without the capacity layout need the same workspace."""
    import ctypes as C

    from paper_2608_11091_amd import _abi, api
    rng = np.random.default_rng(4)
    lib = _abi.load()
    sizes = set()
    for r in ((6, 6, 6), (6, 5, 6), (1, 6, 2)):
        x = tk.Tucker.from_numpy(rng.standard_normal(r), [rng.standard_normal((20, k)) for k in r], rcap=(6, 6, 6))
        bs, keep = api._blocks_struct([(1.0, x), (2.0, x)])
        nb = C.c_size_t()
        api.check(lib.tucker_sketch_workspace(C.byref(bs), 12, 0, C.byref(nb)))
        sizes.add(nb.value)
    assert len(sizes) == 1
