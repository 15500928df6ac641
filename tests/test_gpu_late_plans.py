"""Iterations planned ahead (the first k_trunc) and when they are first enqueued
(the others) run the same work: a cycle limited to m iterations repeats, bit
for bit, the first m residuals and ranks of a longer one, for m below, at and
above k_trunc, in both precisions, and a restarted solve replays its plans."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from workloads import draw_sketches, laplacian_1d  # noqa: E402


@pytest.fixture(scope="module")
def tk():
    import paper_2608_11091_amd as tk
    tk.load()
    return tk


def _cm(M):
    return torch.from_numpy(np.ascontiguousarray(M.T)).cuda()


def _solve(tk, form, k_trunc, maxiter, restarts):
    n, cap, p = 20, 12, 3
    L = laplacian_1d(n)
    op = tk.KronOp.from_terms([(1.0, [L if j == k else None for j in range(3)]) for k in range(3)])
    b = tk.Tucker.from_numpy(np.ones((1, 1, 1)), [np.ones((n, 1))] * 3, rcap=(cap,) * 3)
    S, Om = draw_sketches([n] * 3, 40, cap, p)
    prm = tk.SolveParams(form=form, tol=1e-13, maxiter=maxiter, k_trunc=k_trunc, rank_cap=cap, oversample=p,
                         max_restarts=restarts)
    return tk.solve(op, b, [_cm(a) for a in S], [_cm(a) for a in Om], prm)


@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("k_trunc", [1, 2, 4])
def test_late_plans(tk, form, k_trunc):
    x, long_ = _solve(tk, form, k_trunc, 8, 1)
    for m in (1, k_trunc, k_trunc + 1, 7):
        _, info = _solve(tk, form, k_trunc, m, 1)
        assert info["iters"] == m
        assert np.array_equal(info["hist"], long_["hist"][:m])
        assert info["ranks"] == long_["ranks"][:m]
    x1, two = _solve(tk, form, k_trunc, 5, 2)
    x2, again = _solve(tk, form, k_trunc, 5, 2)
    assert two["cycles"] == 2 and two["iters"] == 10
    assert np.array_equal(two["hist"], again["hist"]) and np.array_equal(two["hist"][:5], long_["hist"][:5])
    assert torch.equal(x1.core, x2.core)
