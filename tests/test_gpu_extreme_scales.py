"""ST-HOSVD eigensolver on Grams at the ends of the exponent range.  The solver
scales its matrix by a power of two; the Gram of a tensor of norm 1e-156 (FP64)
or 2e-20 (FP32, BF16 factors) has a denormal trace, the reciprocal of which
overflows, and that of a tensor of norm 1.2e154 or 1.6e19 a trace in the last
binade.

Tiny tensors: width and ranks are forced to the tensor's own, so the
eigenvectors are a full orthonormal basis whatever the accuracy of the Gram and
the sum is reproduced to rounding: a few hundred operations at 1e-16, 6e-8 or
(factor products of the BF16 form) 4e-3.  Large ones: the width is forced, the
ranks follow the rule, which cuts the rounding behind a tensor of exact rank."""
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


def _case(seed, n, r, norm, w):
    rng = np.random.default_rng(seed)
    core = rng.standard_normal((r,) * 3)
    core *= 1.0 / np.linalg.norm(core)
    X = O.Tucker(core, [np.linalg.qr(rng.standard_normal((n, r)))[0] for _ in range(3)])
    # sketches scaled so that the range sketches have entries of O(1)
    Om = [rng.standard_normal((n, w)) for _ in range(3)]
    f = min(max(1.0 / np.sqrt(norm), 1e-12 if norm > 1 else 1.0), 1e12)
    return X, [torch.from_numpy(np.ascontiguousarray(f * o.T)).cuda() for o in Om]


@pytest.mark.parametrize("form,norm,tol", [(0, 1e-156, 1e-12), (1, 2e-20, 1e-4), (2, 2e-20, 5e-2)])
@pytest.mark.parametrize("n,r", [(24, 5), (40, 16)])
def test_tiny(tk, form, norm, tol, n, r):
    X, om = _case(r, n, r, norm, r)
    t = tk.Tucker.from_numpy(X.core * norm, X.U)
    got, s = tk.rhosvd([(1.0, t)], om, 1e-10 if form == 0 else 1e-5, r, 0, force_s=r, force_ranks=(r,) * 3, form=form)
    core, U = got.to_numpy()
    assert np.isfinite(core).all() and all(np.isfinite(u).all() for u in U)
    dist = O.exact_norm([(1.0, O.Tucker(core / norm, U)), (-1.0, X)])
    orth = max(np.abs(u.T @ u - np.eye(r)).max() for u in U)
    print(f"tiny form {form} n {n} r {r}: dist {dist:.1e} orth {orth:.1e}", flush=True)
    assert dist <= tol and orth <= tol


@pytest.mark.parametrize("form,norm,eps,tol", [(0, 1.2e154, 1e-6, 1e-12), (1, 1.6e19, 1e-3, 1e-4)])
@pytest.mark.parametrize("n,r,p", [(24, 5, 3), (40, 16, 5)])
def test_last_binade(tk, form, norm, eps, tol, n, r, p):
    X, om = _case(10 + r, n, r, norm, r + p)
    t = tk.Tucker.from_numpy(X.core * norm, X.U)
    got, s = tk.rhosvd([(1.0, t)], om, eps, r + p, 0, force_s=r + p, form=form)
    core, U = got.to_numpy()
    assert got.ranks == (r,) * 3
    dist = O.exact_norm([(1.0, O.Tucker(core / norm, U)), (-1.0, X)])
    print(f"last binade form {form} n {n} r {r}: dist {dist:.1e}", flush=True)
    assert dist <= tol
