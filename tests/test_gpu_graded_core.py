"""FP32 and FP64 RoundSums of a superdiagonal core whose last entry is far below
the others: its square, a diagonal entry of the ST-HOSVD Gram, is a denormal of
the form (or just above).  Unit factors and sketches make every intermediate a
diagonal, so the result is the input: factors with orthonormal columns to the
rounding of the form and the core to that rounding of its norm.

The range basis cuts a column whose second-pass pivot, after the first pass's
shift 11 (n s + s (s + 1)) u tr, is at or below 1e-30 of the trace: its basis
column, and the factor column on it, is zero."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def tk():
    import paper_2608_11091_amd as tk
    tk.load()
    return tk


@pytest.mark.parametrize("form,small,tol", [(1, s, 1e-5) for s in (1e-17, 3e-18, 4e-19, 1e-19, 6e-20, 2e-20, 4e-21)] +
                         [(0, s, 1e-13) for s in (1e-8, 1e-19, 4e-21)])
@pytest.mark.parametrize("r", [3, 9, 24])
def test_graded_core(tk, form, small, tol, r):
    n = r + 4
    core = np.zeros((r,) * 3)
    sig = np.linspace(1.0, 0.5, r)
    sig[-1] = small
    i = np.arange(r)
    core[i, i, i] = sig
    eye = torch.from_numpy(np.ascontiguousarray(np.eye(n, r).T)).cuda()
    t = tk.Tucker.from_numpy(core, [np.eye(n, r) for _ in range(3)])
    got, s = tk.rhosvd([(1.0, t)], [eye] * 3, 1e-30, r, 0, force_s=r, force_ranks=(r,) * 3, form=form)
    g, U = got.to_numpy()
    unit = np.ones(r)
    tr = (sig ** 2).sum()
    unit[-1] = small ** 2 / (small ** 2 + 11.0 * (n * r + r * (r + 1)) * 2.0 ** -53 * tr) > 1e-30 * (r - 1)
    orth = max(np.abs(np.sort(u.T @ u, axis=None) - np.sort(np.diag(unit), axis=None)).max() for u in U)
    for u in U:
        g = np.moveaxis(np.tensordot(u, g, axes=([1], [0])), 0, -1)
    ref = np.zeros((n,) * 3)
    ref[i, i, i] = sig
    err = np.abs(g - ref).max()
    print(f"graded form {form} r {r} small {small}: err {err:.1e} orth {orth:.1e}", flush=True)
    assert np.isfinite(g).all() and orth <= tol and err <= tol
