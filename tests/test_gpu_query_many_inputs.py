"""The workspace query of a solve and of its adjoint covers the call for every
number of inputs: the tables of the finiteness check hold one entry per input,
and the query, which is asked without sketches, counted fewer.  Terms and orders
walk the entries over multiples of 32 (one 256-byte step of the workspace)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _problem(tk, d, nterms, n=6):
    rng = np.random.default_rng(10 * d + nterms)
    terms = [(1.0 if j == 0 else 0.01, [2.0 * np.eye(n) + 0.1 * rng.standard_normal((n, n)) for _ in range(d)])
             for j in range(nterms)]
    b = tk.Tucker.from_numpy(rng.standard_normal((2,) * d), [rng.standard_normal((n, 2)) for _ in range(d)])
    cm = lambda w: [torch.from_numpy(rng.standard_normal((w, n))).cuda() for _ in range(d)]
    return tk.KronOp.from_terms(terms), b, cm(20), cm(5)


@pytest.mark.parametrize("d,terms", [(2, range(1, 22)), (3, range(1, 14)), (4, range(1, 10))])
@pytest.mark.parametrize("form", [0, 1])
def test_solve_and_adjoint(d, terms, form):
    import paper_2608_11091_amd as tk
    prm = tk.SolveParams(form=form, tol=1e-2, maxiter=4, max_restarts=1, rank_cap=3, oversample=2)
    for nterms in terms:
        op, b, S, om = _problem(tk, d, nterms)
        print(f"d {d} terms {nterms} form {form}", flush=True)
        for x0 in (None, b):
            x, info = tk.solve(op, b, S, om, prm, x0=x0)
            assert np.isfinite(info["true_relres"])
        lam, dal, dA, info = tk.backward(op, x, [(1.0, x), (-0.5, b)], S, om, prm)
        assert np.isfinite(info["true_relres"]) and np.isfinite(dal).all()
