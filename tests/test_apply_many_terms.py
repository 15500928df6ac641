"""Operators with more than 256 factor products: the workspace query answers for
any number of terms (no GPU needed), and the grouped products are right."""
import ctypes as C
import os

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2608_11091_amd", "libtsgmres.so")


@pytest.mark.skipif(not os.path.exists(LIB), reason="library not built")
@pytest.mark.parametrize("d,nterms", [(4, 64), (4, 65), (4, 400), (3, 86), (2, 129), (2, 5000)])
@pytest.mark.parametrize("form", [0, 1, 2])
def test_query(d, nterms, form):
    from paper_2608_11091_amd import _abi
    op, x = _abi.TkKronOp(), _abi.TkTucker()
    op.d, op.nterms, x.d, x.core = d, nterms, d, 0x1000
    for k in range(d):
        op.n[k], x.n[k], x.r[k], x.rcap[k], x.U[k] = 8, 8, 2, 2, 0x1000
    alpha, A = (C.c_double * nterms)(*[1.0] * nterms), (C.c_void_p * (nterms * d))(*[0x1000] * (nterms * d))
    op.alpha, op.A = alpha, A
    need = C.c_size_t()
    _abi.check(_abi.load().tucker_apply_op_workspace(C.byref(op), C.byref(x), form, C.byref(need)))
    assert need.value > 0


@pytest.mark.gpu
@pytest.mark.parametrize("form,tol", [(0, 1e-13), (1, 1e-5)])
def test_products(form, tol):
    import paper_2608_11091_amd as tk
    rng = np.random.default_rng(3)
    ns, r, nterms = (9, 7, 9), 3, 120
    x = tk.Tucker.from_numpy(rng.standard_normal((r,) * 3), [rng.standard_normal((n, r)) for n in ns])
    terms = [(1.0, [rng.standard_normal((n, n)) for n in ns]) for _ in range(nterms)]
    blocks = tk.apply_op(tk.KronOp.from_terms(terms), x, form=form)
    for (_, As), (_, y) in zip(terms, blocks):
        for k, A in enumerate(As):
            ref = x.U[k].cpu().numpy() @ A.T
            assert np.linalg.norm(y.U[k].cpu().numpy() - ref) <= tol * np.linalg.norm(ref)
