"""Householder QR kernels on nearly triangular columns: e_j plus a part below
the diagonal of norm 8e-9, whose square is lost beside the diagonal's.  The
factorisation must still carry it (backward stability: 1e-16 of the column, not
1e-8), through the calls that run the kernels: the exact norm (R only, plain,
and pivoted for a second block) and the multilinear Nystrom recovery (pivoted
QR with Q).  Row counts walk the kernels' row blocks.  Bounds: a few hundred
operations at 1e-16 for the norms (1e-12), the recovery's 1e-10; the difference
of two columns 8e-9 apart keeps 1e-16 / 8e-9 of itself (1e-6 asserted)."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BELOW = 8e-9


@pytest.fixture(scope="module")
def tk():
    import paper_2608_11091_amd as tk
    tk.load()
    return tk


def _cm(M):
    return torch.from_numpy(np.ascontiguousarray(M.T)).cuda()


def _factor(rng, n, r):
    """Columns e_j with a part of norm BELOW spread over the rows below."""
    E = np.tril(rng.standard_normal((n, r)), -1)
    nrm = np.linalg.norm(E, axis=0)
    return np.eye(n, r) + BELOW * E / np.where(nrm > 0.0, nrm, 1.0)


def _ref_norm(blocks):
    """Norm through the Gram of the factors in extended precision (r small)."""
    total = np.longdouble(0.0)
    for ci, X in blocks:
        for cj, Y in blocks:
            G = [u.astype(np.longdouble).T @ v.astype(np.longdouble) for u, v in zip(X.U, Y.U)]
            Z = Y.core.astype(np.longdouble)
            for k, g in enumerate(G):
                Z = np.moveaxis(np.tensordot(g, Z, axes=([1], [k])), 0, k)
            total += np.longdouble(ci) * np.longdouble(cj) * (X.core.astype(np.longdouble) * Z).sum()
    return float(np.sqrt(total))


@pytest.mark.parametrize("n,r", [(4, 4), (16, 5), (64, 8), (65, 33), (130, 12), (257, 16), (512, 48)])
def test_norm(tk, n, r):
    rng = np.random.default_rng(n + r)
    X = [O.Tucker(rng.standard_normal((r,) * 3), [_factor(rng, n, r) for _ in range(3)]) for _ in range(2)]
    for blocks in ([(1.0, X[0])], [(1.0, X[0]), (-0.5, X[1])]):
        ref = _ref_norm(blocks)
        got = tk.norm([(c, tk.Tucker.from_numpy(x.core, x.U)) for c, x in blocks])
        print(f"norm n {n} r {r} blocks {len(blocks)}: {got / ref - 1.0:.1e}", flush=True)
        assert abs(got / ref - 1.0) <= 1e-12


@pytest.mark.parametrize("n", [2, 64, 65, 300])
def test_norm_of_a_difference(tk, n):
    # (e_1 + 8e-9 e_n) - e_1, within one block and as two blocks
    e1, en = np.eye(n)[:, :1], np.eye(n)[:, n - 1:]
    U = np.concatenate([e1 + BELOW * en, e1], axis=1)
    one = [(1.0, O.Tucker(np.array([[1.0], [-1.0]]), [U, e1]))]
    two = [(1.0, O.Tucker(np.ones((1, 1)), [U[:, :1], e1])), (-1.0, O.Tucker(np.ones((1, 1)), [e1, e1]))]
    for blocks in (one, two):
        got = tk.norm([(c, tk.Tucker.from_numpy(x.core, x.U)) for c, x in blocks])
        print(f"difference n {n} blocks {len(blocks)}: {got / BELOW - 1.0:.1e}", flush=True)
        assert abs(got / BELOW - 1.0) <= 1e-6


@pytest.mark.parametrize("n,r", [(12, 4), (64, 16), (100, 20), (200, 12)])
def test_recovery(tk, n, r):
    # Psi = I: the core sketch is the tensor, P_k the projector onto range(F_k)
    rng = np.random.default_rng(n * r)
    X = O.Tucker(rng.standard_normal((r,) * 3), [_factor(rng, n, r) for _ in range(3)])
    dense = X.core
    for k, u in enumerate(X.U):
        dense = np.moveaxis(np.tensordot(u, dense, axes=([1], [k])), 0, k)
    got = tk.mln_recover(torch.from_numpy(np.ascontiguousarray(dense)).cuda(), [_cm(u) for u in X.U],
                         [_cm(np.eye(n)) for _ in range(3)], r)
    core, U = got.to_numpy()
    for k, u in enumerate(U):
        core = np.moveaxis(np.tensordot(u, core, axes=([1], [k])), 0, k)
    dist = np.linalg.norm(core - dense) / np.linalg.norm(dense)
    print(f"recovery n {n} r {r}: ranks {got.ranks} dist {dist:.1e}", flush=True)
    assert got.ranks == (r,) * 3
    assert dist <= 1e-10
