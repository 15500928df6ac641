"""Effective-rank rule, FP64, at its zero clamp delta = 1e-12 of the largest
eigenvalue.  A block with two dyadic columns and one with a unit column have a
Gram that FP64 holds exactly and that is tridiagonal as it stands, with
lambda_1 inside its Gershgorin interval and one eigenvalue a given share above
or below the clamp; whether this one counts moves the width by one.  (tau is far
below the clamp: the rank is the number of eigenvalues above it.)"""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [8, 40, 64, 100])
@pytest.mark.parametrize("share", [1e-6, 1e-8, 1e-10, 1e-11, 1e-12])
@pytest.mark.parametrize("side", [1.0, -1.0])
def test_clamp(n, share, side):
    import paper_2608_11091_amd as tk
    rng = np.random.default_rng(n)
    cap, p = 6, 2
    om = [torch.from_numpy(rng.standard_normal((cap + p, n))).cuda() for _ in range(3)]
    e = np.eye(n)
    got = []
    for a, b in [(0.5, 0.25), (0.25, 0.75), (0.75, 1.5), (1.25, 0.5), (0.125, 1.0), (1.75, 0.875)]:
        U = np.zeros((n, 2))
        U[0], U[1, 1] = (1.0, a), b
        # w^2 = 4 (a core of four ones has norm 2, exactly)
        tr, det = np.longdouble(1 + a * a + b * b), np.longdouble(b * b)
        lam = 4 * (tr / 2 + np.sqrt(tr * tr / 4 - det))
        small = float(np.sqrt(np.longdouble(1e-12) * lam * (1 + np.longdouble(side * share))))
        core = np.zeros((2, 2, 2))
        core[0, 0, 0] = core[0, 1, 1] = core[1, 0, 1] = core[1, 1, 0] = 1.0
        blocks = [(1.0, O.Tucker(core, [U] * 3)), (small, O.Tucker(np.ones((1,) * 3), [e[:, 2:3]] * 3))]
        got.append(tk.rhosvd([(c, tk.Tucker.from_numpy(X.core, X.U)) for c, X in blocks], om, 1e-10, cap, p)[1])
    print(f"n {n} share {side * share}: s {got}", flush=True)
    assert got == [2 + p + (1 if side > 0 else 0)] * 6
